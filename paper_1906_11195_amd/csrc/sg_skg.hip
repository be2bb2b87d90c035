// Sherrington-Kirkpatrick sweeps with real couplings (Eq. 1: Gaussian J_ij
// of variance 1/N, given as float32) on gfx950.
//
// The local fields h_i = sum_j J_ij s_j are real and are kept in IEEE double.
// A flip of s_i changes every field by 2 s_i J_ij (new s_i): the product is
// exact in double, so a field's value depends only on the order in which the
// flips reach it, and this kernel applies them to every field in flip order,
// as the sequential definition does.  Every `period` sweeps the fields are
// recomputed directly (skg_recompute below), which bounds the rounding drift of
// the incremental sums (SI, SK section: the force is the costly part and is
// recomputed periodically).
//
// Acceptance of a move with x = s_i h_i: x <= 0 accepts, else the move is
// accepted iff r < floor(ldexp(exp(-beta (2 x)), 32)) in double, r the same
// 32-bit uniform as for binary couplings.
//
// One workgroup runs one chain, visiting i = 0..N-1 in blocks of 64 spins, as a
// pipeline of roles over the blocks (block g of the launch):
//
//  * prep wavefronts (two): load the block's two 64 x 64 coupling tiles straight
//    into LDS (rows of the block's own spins and of the block before it, its
//    columns) and draw the uniforms and their bounds on x.
//  * decider wavefront: lane i owns spin 64 b + i.  It takes the block's fields
//    as published after block g - 2, adds the flips of block g - 1 in order, and
//    finds the flips as a fixpoint: each round it adds the last guess's flips, in
//    order, to the fields of the lanes after them (from the tile) and tests every
//    lane.  A lane's test depends on lanes before it only, so the fixpoint is
//    unique, is the sequential result, and is reached in two or three rounds.
//    A round leaves the list of its flips in LDS, in order.
//  * updater wavefronts (thirteen): a lane keeps V consecutive fields per item of
//    64 V in registers (item w, w + 13, ... for wavefront w; V = 4, less for small
//    N so that more wavefronts share the work), reads the flipped spins' rows, up
//    to 8 flips of an item at a time, and adds them in order; then it publishes the
//    fields of the block after next if it has them.
//
// Rows are padded to whole items (skg_pitch), so that every row starts 16-byte
// aligned whatever N is and no item has a tail.
//
// What bounds it: the chain updaters -> decider -> updaters.  A block's rows (4 N
// bytes a flip, 6.4 flips a block) are asked for once it is decided, and take a
// memory latency and their transfer (one CU takes in about 90 GB/s); the decider
// is at the next block meanwhile, about 1 us for its two or three rounds.  A block
// takes 1.24 us at N = 1021, 1.70 at 4096 and 2.96 when the couplings of all
// samples exceed the 256 MiB of the memory-side cache (32 samples of 4096); 4.4,
// 5.4 and 5.4 us with the roles in turn, a workgroup barrier after each, as before.
// Measured and dropped: asking for the next block's rows before adding this one's
// (the decider is not done with it: 1.5 and 2.0 us, 3.0 where memory is the bound),
// a wavefront that touches the rows in advance (2.3 and 3.8 us: its line by line
// reads take the loads' place).
#include <type_traits>

#include "sg_internal.h"
#include "sg_philox.h"
#include "sg_pipe.h"

namespace sg {
namespace {

typedef double v2d __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

constexpr int kSlots = 3;           // blocks whose tiles and bounds are in LDS
constexpr int kHRing = 4;           // published fields of coming blocks
constexpr int kLRing = 128;         // flip lists of past blocks (an updater's blocks are at most 104 apart)
constexpr int kLst = 72;            // entries of a list: 64, and fillers up to a whole batch
constexpr int kBatch = 8;           // flips taken at a time
constexpr int kPrep = 2;
constexpr int kUpd = 13;
constexpr int kSkgThreads = 64 * (1 + kPrep + kUpd);
constexpr uint32_t kTile = 65 * 256;   // bytes of a tile: 64 rows of 64 floats and a row of zeros
// An entry of the decider's own lists (16 bits): flipped lane << 8 (a row's offset
// in a tile) | (new spin -1) << 15; kNoFlip is none (the row of zeros).  The
// updaters' entries: offset of the row from the block's first one | (new spin -1)
// << 31.
constexpr uint32_t kNoFlip = 64u << 8;

struct SkgLds {
    uint32_t tile;    // [kSlots][2] tiles: rows of the block, rows of the block before
    uint32_t bnd;     // [kSlots][64] double lo, hi: acceptance bounds (SkgBound)
    uint32_t rnd;     // [kSlots][64] uniforms
    uint32_t hr;      // [kHRing][64] doubles: published fields
    uint32_t own;     // uint16 [2][kLst]: flips of a block in lane order, then fillers (the decider's)
    uint32_t list;    // uint32 [kLRing][64]: flips of past blocks (the updaters')
    uint32_t cnt;     // [kLRing] their numbers
    uint32_t bits;    // uint64 [NB]: spins, bit 1 = -1
    uint32_t seqp;    // [kSlots] 1 + block whose tiles and bounds are in the slot
    uint32_t seqh;    // [kHRing] 1 + block whose fields are in the slot
    uint32_t sync;    // blocks decided, abort
    uint32_t total;
};

__host__ __device__ __forceinline__ SkgLds skg_layout(int32_t n)
{
    SkgLds L;
    uint32_t off = 0;
    auto take = [&](uint32_t bytes) {
        const uint32_t p = off;
        off += (bytes + 15u) & ~15u;
        return p;
    };
    L.tile = take(kSlots * 2 * kTile);
    L.bnd = take(kSlots * 64 * 16);
    L.rnd = take(kSlots * 64 * 4);
    L.hr = take(kHRing * 64 * 8);
    L.own = take(2 * kLst * 2);
    L.list = take(kLRing * 64 * 4);
    L.cnt = take(kLRing * 4);
    L.bits = take((uint32_t)((n + 63) >> 6) * 8u);
    L.seqp = take(kSlots * 4);
    L.seqh = take(kHRing * 4);
    L.sync = take(8);
    L.total = off;
    return L;
}

// Waits until `target` blocks of the launch are decided.
__device__ __forceinline__ void wait_decided(uint32_t sync, int32_t target)
{
    int spins = 0;
#pragma unroll 1
    while (__builtin_amdgcn_readfirstlane(lds_get<int32_t>(sync)) < target) {
        if (wait_giveup(sync, spins)) return;
        __builtin_amdgcn_s_sleep(1);
    }
}

__device__ __forceinline__ bool skg_accept(double x, double beta, uint32_t r)
{
    if (x <= 0.0) return true;
    const double p = exp(-beta * (2.0 * x));
    const uint64_t thr = (uint64_t)floor(ldexp(p, 32));
    return (uint64_t)r < thr;
}

// The same decision through a per-lane bound on x, fixed by r before the
// rounds: r < floor(2^32 exp(-2 beta x)) holds iff 2^32 exp(-2 beta x) >=
// r + 1, i.e. x <= xc = -ln((r + 1) 2^-32) / (2 beta).  Outside a band of
// relative width 1e-9 around xc (far wider than the rounding of exp, ln and
// the division) the bound decides; inside it the rule itself does, so every
// decision is that of skg_accept.  `lo` is at least the smallest positive
// number, so that x < lo holds for every x <= 0.
struct SkgBound {
    double lo, hi;   // accept below lo, reject above hi, else evaluate
};

__device__ __forceinline__ SkgBound skg_bound(double beta, uint32_t r)
{
    constexpr double kTiny = 4.9406564584124654e-324;
    if (beta == 0.0) return SkgBound{HUGE_VAL, HUGE_VAL};      // threshold 2^32: every move
    if (beta > 1.7976931348623157e308) return SkgBound{kTiny, 0.0};   // threshold 0: none with x > 0
    if (!(beta < 1e300)) return SkgBound{kTiny, HUGE_VAL};
    const double xc = -log(((double)r + 1.0) * 0x1p-32) / (2.0 * beta);
    const double band = 1e-9 * (xc + 1.0);
    return SkgBound{xc - band > kTiny ? xc - band : kTiny, xc + band};
}

// ---------------- prep ----------------
__device__ __forceinline__ void skg_prep(const SkChain* ch, const SkgLds& L, uint32_t lds, int pw, int64_t t0,
                                         int32_t total)
{
    const int lane = threadIdx.x & 63;
    const int32_t n = ch->n, NB = (n + 63) >> 6, np = skg_pitch(n);
    const uint64_t seed = ch->seed;
    const uint32_t rep = ch->rep, inst = ch->inst;
    const double beta = ch->beta;
    const SG_G float* J = gl(ch->Jf);
    const SG_G float* Jd = gl(ch->Jd) + lane * 4;
    int32_t b = pw % NB, s = pw / NB, slot = pw % kSlots;
    for (int32_t g = pw; g < total; g += kPrep) {
        if (g >= kSlots) wait_decided(lds + L.sync, g - kSlots + 1);
        // both tiles, 1 KiB (4 rows) a load, straight to LDS
        const uint32_t to = lds + L.tile + (uint32_t)slot * 2u * kTile;
        const int32_t rb = (b == 0 ? NB : b) * 64 - 64;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            __builtin_amdgcn_global_load_lds((const SG_G void*)(Jd + (int64_t)b * 4096 + q * 256),
                                             (SG_L void*)(size_t)(to + q * 1024), 16, 0, 0);
            const int32_t row = min(rb + 4 * q + (lane >> 4), n - 1);   // (rows past n are not used)
            __builtin_amdgcn_global_load_lds((const SG_G void*)(J + (int64_t)row * np + b * 64 + (lane & 15) * 4),
                                             (SG_L void*)(size_t)(to + kTile + q * 1024), 16, 0, 0);
        }
        // the acceptance uniforms of the block's positions (the two half-word
        // streams of the binary model, both drawn) and their bounds
        const uint32_t p = (uint32_t)(b * 64 + lane), t = (uint32_t)(t0 + s);
        const U4 A = philox_stream(seed, p >> 3, t, kDomSweepHi, rep, inst);
        const U4 B = philox_stream(seed, p >> 3, t, kDomSweepLo, rep, inst);
        const uint32_t r = (half_word(A, p & 7u) << 16) | half_word(B, p & 7u);
        const SkgBound bd = skg_bound(beta, r);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the tiles are in LDS
        const bool act = (int32_t)p < n;                   // (a lane past the last spin never flips)
        lds_put<v2d>(lds + L.bnd + (uint32_t)(slot * 64 + lane) * 16u,
                     v2d{act ? bd.lo : -HUGE_VAL, act ? bd.hi : -HUGE_VAL});
        lds_put<uint32_t>(lds + L.rnd + (uint32_t)(slot * 64 + lane) * 4u, r);
        if (lane == 0) lds_put<int32_t>(lds + L.seqp + 4u * (uint32_t)slot, g + 1);
        slot += kPrep;
        if (slot >= kSlots) slot -= kSlots;
        for (b += kPrep; b >= NB; b -= NB) ++s;
    }
}

// ---------------- decider ----------------
__device__ __forceinline__ void skg_decide(const SkChain* ch, const SkgLds& L, uint32_t lds, int64_t t0, int32_t total,
                                           int64_t t_max)
{
    __builtin_amdgcn_s_setprio(3);   // the sequential critical path
    const int lane = threadIdx.x & 63;
    const int32_t n = ch->n, NB = (n + 63) >> 6, wn = ch->words_n;
    const double beta = ch->beta;
    unsigned long long acc = 0;
    const uint32_t lofs = lds + L.tile + 4u * (uint32_t)lane;
    const uint32_t urow = (uint32_t)lane * (uint32_t)skg_pitch(n) * 4u;
    // h + the flips of a list entry pair w, in order: a 2 s' J product is exact,
    // so the fused operation rounds as the sum alone
    auto add2 = [&](double h, uint32_t w, float v0, float v1) {
        const double a0 = __hiloint2double((int)(((w << 16) & 0x80000000u) | 0x40000000u), 0);
        const double a1 = __hiloint2double((int)((w & 0x80000000u) | 0x40000000u), 0);
        return fma(a1, (double)v1, fma(a0, (double)v0, h));
    };
    auto add8 = [&](double h, v4u w, uint32_t tile) {
        const uint32_t e[4] = {w.x, w.y, w.z, w.w};
        float v[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] = *(const SG_L float*)(size_t)(tile + (e[i] & 0x7f00u));
            v[2 * i + 1] = *(const SG_L float*)(size_t)(tile + ((e[i] >> 16) & 0x7f00u));
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) h = add2(h, e[i], v[2 * i], v[2 * i + 1]);
        return h;
    };
    int32_t b = 0, s = 0, slot = 0;
    int32_t pnf = 0;              // flips of the block before, the first 8 of them
    v4u pw = v4u{0u, 0u, 0u, 0u};
    for (int32_t g = 0; g < total; ++g) {
        const uint32_t hs = (uint32_t)g & (kHRing - 1);
        int32_t sp, sh;
        double h;
        v2d bd;
        int spins = 0;
        for (;;) {
            sp = lds_get<int32_t>(lds + L.seqp + 4u * (uint32_t)slot);
            sh = lds_get<int32_t>(lds + L.seqh + 4u * hs);
            h = lds_get<double>(lds + L.hr + (hs * 64u + (uint32_t)lane) * 8u);
            bd = lds_get<v2d>(lds + L.bnd + (uint32_t)(slot * 64 + lane) * 16u);
            if (__builtin_amdgcn_readfirstlane((sp ^ (g + 1)) | (sh ^ (g + 1))) == 0) break;
            if (wait_giveup(lds + L.sync, spins)) break;
        }
        const unsigned long long SB = ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane(
                                           lds_get<int32_t>(lds + L.bits + 8u * (uint32_t)b + 4u)) << 32) |
                                      (uint32_t)__builtin_amdgcn_readfirstlane(lds_get<int32_t>(lds + L.bits + 8u * (uint32_t)b));
        const uint32_t neg = __builtin_amdgcn_inverse_ballot_w64(SB) ? 0x80000000u : 0u;
        const uint32_t own = lofs + (uint32_t)slot * 2u * kTile, prev = own + kTile;
        // the flips of the block before
        if (pnf > 0) h = add8(h, pw, prev);
        for (int32_t f = kBatch; f < pnf; f += kBatch)
            h = add8(h, lds_get<v4u>(lds + L.own + (((uint32_t)g - 1u) & 1u) * (kLst * 2) + 2u * (uint32_t)f), prev);
        auto test = [&](double hc) -> unsigned long long {
            const double x = __hiloint2double(__double2hiint(hc) ^ (int)neg, __double2loint(hc));
            const unsigned long long a = __builtin_amdgcn_ballot_w64(x < bd.x);
            const unsigned long long u = __builtin_amdgcn_ballot_w64(x <= bd.y) & ~a;
            if (u == 0ull) return a;
            // inside the band around a lane's bound: the rule itself
            bool f = false;
            if ((u >> lane) & 1ull) f = skg_accept(x, beta, lds_get<uint32_t>(lds + L.rnd + (uint32_t)(slot * 64 + lane) * 4u));
            return a | __builtin_amdgcn_ballot_w64(f);
        };
        const uint32_t lst = lds + L.own + ((uint32_t)g & 1u) * (kLst * 2);
        const uint32_t ring = (uint32_t)g & (kLRing - 1);
        uint32_t rank = 0u;
        unsigned long long F = test(h);
        int32_t nf = 0;
        v4u w = v4u{0u, 0u, 0u, 0u};
        while (F != 0ull) {
            // the list of F in lane order, fillers after it
            nf = __popcll(F);
            rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(F >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)F, 0u));
            const bool mine = __builtin_amdgcn_inverse_ballot_w64(F);
            const uint32_t pos = mine ? rank : (uint32_t)nf + (uint32_t)lane - rank;
            // (the new spin is -1 where the spin is +1)
            const uint32_t ent = mine ? ((uint32_t)lane << 8) | (neg ? 0u : 0x8000u) : kNoFlip;
            lds_put<uint16_t>(lst + 2u * pos, (uint16_t)ent);
            w = lds_get<v4u>(lst);
            double hc = add8(h, w, own);
            for (int32_t f = kBatch; f < nf; f += kBatch) hc = add8(hc, lds_get<v4u>(lst + 2u * (uint32_t)f), own);
            const unsigned long long F2 = test(hc);
            if (F2 == F) break;
            F = F2;
        }
        if (F == 0ull) nf = 0;
        if (__builtin_amdgcn_inverse_ballot_w64(F))
            lds_put<uint32_t>(lds + L.list + (ring * 64u + rank) * 4u, urow | (neg ^ 0x80000000u));
        const unsigned long long SN = SB ^ F;
        if (lane == 0) {
            lds_put<int32_t>(lds + L.cnt + 4u * ring, nf);
            lds_put<uint32_t>(lds + L.bits + 8u * (uint32_t)b, (uint32_t)SN);
            lds_put<uint32_t>(lds + L.bits + 8u * (uint32_t)b + 4u, (uint32_t)(SN >> 32));
            lds_put<int32_t>(lds + L.sync, g + 1);
        }
        pnf = nf;
        pw = w;
        acc += (unsigned long long)nf;
        if (++slot == kSlots) slot = 0;
        if (++b == NB) {
            b = 0;
            ++s;
            const int64_t tn = t0 + s;
            if (tn <= t_max && (tn & (tn - 1)) == 0) {
                const int k = 1 + (63 - __clzll((unsigned long long)tn));
                for (int32_t q = lane; q < wn; q += 64)
                    gl(ch->snap)[(int64_t)k * wn + q] = lds_get<uint32_t>(lds + L.bits + 4u * (uint32_t)q);
            }
        }
    }
    for (int32_t q = lane; q < wn; q += 64) gl(ch->state)[q] = lds_get<uint32_t>(lds + L.bits + 4u * (uint32_t)q);
    if (lane == 0 && acc) atomicAdd(ch->accepted, acc);
}

// ---------------- updaters ----------------
template <int V>
struct SkgVec;
template <>
struct SkgVec<1> {
    typedef float type;
    static __device__ __forceinline__ float at(type v, int) { return v; }
};
template <>
struct SkgVec<2> {
    typedef float type __attribute__((ext_vector_type(2)));
    static __device__ __forceinline__ float at(type v, int c) { return v[c]; }
};
template <>
struct SkgVec<4> {
    typedef float type __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ float at(type v, int c) { return v[c]; }
};

template <int V, int NI>
__device__ __forceinline__ void skg_update(const SkChain* ch, const SkgLds& L, uint32_t lds, int uw, int32_t total)
{
    typedef typename SkgVec<V>::type vec;
    constexpr int kItem = 64 * V;
    const int lane = threadIdx.x & 63;
    const int32_t n = ch->n, NB = (n + 63) >> 6, nit = (n + kItem - 1) / kItem;
    const uint32_t pitch = (uint32_t)skg_pitch(n) * 4u;   // bytes of a row
    if (uw >= nit) return;
    double h[NI][V];
    const SG_G double* Hd = gl(ch->Hd);
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int c = 0; c < V; ++c) {
            const int32_t i = (uw + kUpd * j) * kItem + V * lane + c;
            h[j][c] = i < n ? Hd[i] : 0.0;
        }
    const uint64_t J = (uint64_t)ch->Jf + (uint32_t)(uw * kItem * 4);
    // A batch: flips f0 .. f0 + kB - 1 of block k (index b, nf flips): their rows'
    // offsets and the high words of their factors 2 s' (the low words are 0), which
    // a lane works out for flip lane & 7.
    int32_t k = 0, b = 0, f0 = 0, nf = 0;
    int32_t pb = 2 % NB;   // block whose fields are published next
    int32_t dec, cnt;
    uint32_t ent;
    auto look = [&]() __attribute__((always_inline)) {
        const uint32_t ring = (uint32_t)k & (kLRing - 1);
        dec = lds_get<int32_t>(lds + L.sync);
        cnt = lds_get<int32_t>(lds + L.cnt + 4u * ring);
        ent = lds_get<uint32_t>(lds + L.list + (ring * 64u + (uint32_t)f0 + ((uint32_t)lane & 7u)) * 4u);
    };
    constexpr int kB = NI > 2 ? 4 : 8;   // (many items: their fields take the registers)
    uint32_t row[kB], ahi[kB];
    auto decode = [&]() __attribute__((always_inline)) {
        const uint32_t last = (uint32_t)(n - 1 - 64 * b) * pitch;   // (no row past the last whatever the entry)
        const uint32_t r = min(ent & 0x7fffffffu, last);
        const uint32_t a = 0x40000000u | (ent & 0x80000000u);
#pragma unroll
        for (int i = 0; i < kB; ++i) {
            row[i] = (uint32_t)__builtin_amdgcn_readlane((int)r, i);
            ahi[i] = (uint32_t)__builtin_amdgcn_readlane((int)a, i);
        }
    };
    // a unit: the batch's rows of one item, two units in flight
    vec v[2][kB];
    auto ask = [&](int j) __attribute__((always_inline)) {
        // (slots past the last item repeat the first one's)
        uint64_t base = J + (uint64_t)((uint32_t)b * 64u * pitch) + (uint64_t)(uw + kUpd * j < nit ? j * kUpd * kItem * 4 : 0);
        uint32_t lo = 4u * V * (uint32_t)lane;
        asm("" : "+s"(base), "+v"(lo));   // (a scalar base and one lane offset: no address arithmetic per lane)
#pragma unroll
        for (int i = 0; i < kB; ++i)
            if (f0 + i < nf) v[j & 1][i] = *(const SG_G vec*)((const SG_G char*)base + (lo + row[i]));
        __builtin_amdgcn_sched_barrier(0);   // (all asked for before any is waited for)
    };
    auto add = [&](int j) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kB; ++i) {
            if (f0 + i >= nf) break;
            const double a = __hiloint2double((int)ahi[i], 0);
#pragma unroll
            for (int c = 0; c < V; ++c) h[j][c] = fma(a, (double)SkgVec<V>::at(v[j & 1][i], c), h[j][c]);
        }
    };
    for (; k < total; ++k) {
        int spins = 0;
        f0 = 0;
#pragma unroll 1
        for (;;) {
            look();
            if (__builtin_amdgcn_readfirstlane(dec) > k) break;
            if (wait_giveup(lds + L.sync, spins)) break;
        }
        nf = __builtin_amdgcn_readfirstlane(cnt);
        while (f0 < nf) {
            decode();
            ask(0);
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                if (j + 1 < NI) ask(j + 1);
                add(j);
            }
            f0 += kB;
            if (f0 < nf) look();
        }
        // the fields of block k + 2
        const int32_t g = k + 2, it = pb / V, js = it / kUpd;
        if (it - js * kUpd == uw && g < total) {
            const uint32_t hs = (uint32_t)g & (kHRing - 1);
            double o[V];
#pragma unroll
            for (int c = 0; c < V; ++c) {
                o[c] = h[0][c];
#pragma unroll
                for (int j = 1; j < NI; ++j) {
                    o[c] = js == j ? h[j][c] : o[c];
                    asm("" : "+v"(o[c]));   // (selects, not an indexed read)
                }
            }
            if (lane / (64 / V) == pb % V) {
                const uint32_t at = lds + L.hr + (hs * 64u + V * ((uint32_t)lane % (64 / V))) * 8u;
#pragma unroll
                for (int c = 0; c < V; ++c) lds_put<double>(at + 8u * c, o[c]);
            }
            if (lane == 0) lds_put<int32_t>(lds + L.seqh + 4u * hs, g + 1);
        }
        if (++pb == NB) pb = 0;
        if (++b == NB) b = 0;
    }
    SG_G double* Ho = gl(ch->Hd);
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int c = 0; c < V; ++c) {
            const int32_t i = (uw + kUpd * j) * kItem + V * lane + c;
            if (i < n) Ho[i] = h[j][c];
        }
}

template <int V, int NI>
__global__ void __launch_bounds__(kSkgThreads) skg_sweep_kernel(const SkChain* __restrict__ chains, int64_t t0,
                                                                int32_t nsw, int64_t t_max, int* err)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t skg_smem[];
    const SkChain* ch = (const SkChain*)(gl(chains) + chain_of_block(blockIdx.x, gridDim.x));
    const uint32_t lds = (uint32_t)(size_t)(SG_L uint8_t*)skg_smem;
    const int32_t n = ch->n, wn = ch->words_n, NB = (n + 63) >> 6;
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const SkgLds L = skg_layout(n);
    const int32_t total = nsw * NB;   // (bounded by the host)
    const SG_G uint32_t* gst = gl(ch->state);
    const SG_G double* Hd = gl(ch->Hd);
    for (int32_t w = tid; w < 2 * NB; w += nthr) lds_put<uint32_t>(lds + L.bits + 4u * (uint32_t)w, w < wn ? gst[w] : 0u);
    // the fields of the first two blocks, which no flip precedes by more than a block
    if (tid < 128) {
        const int32_t i = (tid >> 6) % NB * 64 + (tid & 63);
        lds_put<double>(lds + L.hr + 8u * (uint32_t)tid, i < n ? Hd[i] : 0.0);
    }
    // rows of zeros after the tiles, fillers after the lists
    for (int i = tid; i < kSlots * 2 * 64; i += nthr)
        lds_put<uint32_t>(lds + L.tile + (uint32_t)(i >> 6) * kTile + 64u * 256u + 4u * (uint32_t)(i & 63), 0u);
    if (tid < 2 * (kLst - 64))
        lds_put<uint16_t>(lds + L.own + (uint32_t)(tid / (kLst - 64)) * (kLst * 2) + 2u * (uint32_t)(64 + tid % (kLst - 64)),
                          (uint16_t)kNoFlip);
    if (tid < kLRing) lds_put<int32_t>(lds + L.cnt + 4u * (uint32_t)tid, 0);
    if (tid < kSlots) lds_put<int32_t>(lds + L.seqp + 4u * (uint32_t)tid, 0);
    if (tid < kHRing) lds_put<int32_t>(lds + L.seqh + 4u * (uint32_t)tid, tid < 2 ? tid + 1 : 0);
    if (tid < 2) lds_put<int32_t>(lds + L.sync + 4u * (uint32_t)tid, 0);
    __syncthreads();
    // wavefronts go to the four SIMDs in turn: the decider's SIMD has the prep
    // and one updater, the other three four updaters each
    if (wave == 0)
        skg_decide(ch, L, lds, t0, total, t_max);
    else if (wave == 4 || wave == 8)
        skg_prep(ch, L, lds, (wave >> 2) - 1, t0, total);
    else {
        // (a wavefront with one item less does not read for it)
        const int uw = wave < 12 ? wave - 1 - (wave >> 2) : wave - 3;
        if (NI == 1 || (uw + kUpd * (NI - 1)) * 64 * V < n)
            skg_update<V, NI>(ch, L, lds, uw, total);
        else
            skg_update<V, (NI > 1 ? NI - 1 : 1)>(ch, L, lds, uw, total);
    }
    __syncthreads();
    if (tid == 0 && lds_get<int32_t>(lds + L.sync + 4)) atomicOr(err, 2);
}

// The strict upper triangles of the diagonal tiles: Jd[block][row][column],
// column > row, zero elsewhere (a flip changes the fields of the lanes after it
// within its block).  grid = (blocks, samples); samples that share a matrix write the
// same tiles
__global__ void __launch_bounds__(256) skg_diag_kernel(const SkSample* __restrict__ samples,
                                                       const SkChain* __restrict__ chains)
{
    const SkSample* sm = samples + blockIdx.y;
    const int32_t b = blockIdx.x, n = sm->n, np = skg_pitch(n);
    if (b * 64 >= n) return;
    const float* J = sm->Jf;
    float* Jd = chains[sm->chain0].Jd;
    for (int32_t i = threadIdx.x; i < 4096; i += blockDim.x) {
        const int32_t r = i >> 6, c = i & 63;
        Jd[(int64_t)b * 4096 + i] = c > r && b * 64 + c < n ? J[(int64_t)(b * 64 + r) * np + b * 64 + c] : 0.0f;
    }
}

// ---------------- direct sums ----------------
// A wavefront takes 8 rows of J, 256 columns (16-byte loads) at a time, and the
// block's four wavefronts share the spins of the columns, staged in LDS as bits.
// 32 samples of N = 4096 (2.1 GB of couplings), 2 chains: fields 0.39 ms (5.5 TB/s),
// 16 to 20 snapshots 0.8 to 1.1 ms (arithmetic in double); 1.26 and 2.5 to 3.6 ms
// with one row of 4-byte loads at a time, each row read once per chain and once per
// 8 snapshots, and 0.12 ms for adding the partial sums one after another (now
// 0.005).  6 x 2 chains of N = 1021: 10 and 25 us, before 155 and 240.
constexpr int kRows = 8;
constexpr int kDirect = 256;                        // threads
constexpr int kRowsBlk = kRows * (kDirect / 64);    // rows of a block
constexpr int kCols = 16;                           // snapshots taken at once by skg_bond_kernel

typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double flip_sign(double v, uint32_t m)
{
    return __hiloint2double(__double2hiint(v) ^ (int)m, __double2loint(v));
}

// Sums a[0 .. 15] over the wavefront, in a fixed order: each step halves the values
// a lane carries (17 exchanges; 96 if each value were summed by itself).  Lane l
// gets the sum of value sum_index(l).
__device__ __forceinline__ double wave_sum16(double* a)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int s = 32, cnt = 8; cnt >= 1; s >>= 1, cnt >>= 1) {
        const bool up = (lane & s) != 0;
#pragma unroll
        for (int i = 0; i < cnt; ++i) {
            const double keep = up ? a[i + cnt] : a[i], give = up ? a[i] : a[i + cnt];
            a[i] = keep + __shfl_xor(give, s);
        }
    }
    double v = a[0];
    v += __shfl_xor(v, 2);
    v += __shfl_xor(v, 1);
    return v;
}
// the value whose sum lane l holds (l & 3: copies)
__device__ __forceinline__ int sum_index(int lane) { return lane >> 2; }

// Direct fields h = J s of every chain of one sample, in a fixed order (columns by
// lanes in steps of 256, then wave_sum16), in double; with `check`, a field that
// differs from the incremental one by more than 1e-9 (1 + |h|) raises bit 0 of the
// error word (the rounding drift of a period is many orders of magnitude below
// that).  Two chains share each read of a row; bound by the couplings' bytes.
// grid = (blocks of 32 rows, samples).
__global__ void __launch_bounds__(kDirect) skg_recompute_kernel(const SkSample* __restrict__ samples,
                                                                const SkChain* __restrict__ chains, int check,
                                                                int* err)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t skg_bits[];   // [2][np / 32]
    const SkSample* sm = (const SkSample*)(gl(samples) + blockIdx.y);
    const int32_t n = sm->n, np = skg_pitch(n), nw = np >> 5, wn = (n + 31) >> 5;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if ((int32_t)blockIdx.x * kRowsBlk >= n) return;
    const int32_t i0 = (int32_t)blockIdx.x * kRowsBlk + wave * kRows;
    const SG_G float* J = gl(sm->Jf) + 4 * lane;
    for (int32_t c0 = 0; c0 < sm->nch; c0 += 2) {
        const int nc = min(2, sm->nch - c0);
        const SkChain* ch = (const SkChain*)(gl(chains) + sm->chain0 + c0);
        __syncthreads();
        for (int32_t w = threadIdx.x; w < 2 * nw; w += kDirect) {
            const int c = w >= nw ? 1 : 0;
            const int32_t q = w - c * nw;
            skg_bits[w] = c < nc && q < wn ? gl(ch[c].state)[q] : 0u;
        }
        __syncthreads();
        double acc[2 * kRows];
#pragma unroll
        for (int i = 0; i < 2 * kRows; ++i) acc[i] = 0.0;
        for (int32_t q = 0; q < np; q += 256) {
            v4f v[kRows];
#pragma unroll
            for (int r = 0; r < kRows; ++r) v[r] = *(const SG_G v4f*)(J + (int64_t)min(i0 + r, n - 1) * np + q);
            uint32_t m[2][4];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const uint32_t nib = skg_bits[c * nw + (q >> 5) + (lane >> 3)] >> (4 * (lane & 7));
#pragma unroll
                for (int e = 0; e < 4; ++e) m[c][e] = (nib << (31 - e)) & 0x80000000u;
            }
#pragma unroll
            for (int r = 0; r < kRows; ++r)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double x = (double)v[r][e];
                    acc[r] += flip_sign(x, m[0][e]);
                    acc[kRows + r] += flip_sign(x, m[1][e]);
                }
        }
        const double h = wave_sum16(acc);
        const int idx = sum_index(lane), c = idx / kRows;
        const int32_t i = i0 + idx % kRows;
        if ((lane & 3) == 0 && c < nc && i < n) {
            SG_G double* Hd = gl(ch[c].Hd);
            if (check && fabs(Hd[i] - h) > 1e-9 * (1.0 + fabs(h))) atomicOr(err, 1);
            Hd[i] = h;
        }
    }
}

// Bond sums B = (1/2) sum_i s_i (J s)_i of every snapshot (chain c, grid time
// k) of one sample, in double and in a fixed order: each block forms partial sums
// over 32 rows, written to part[sample][column][block], then skg_bond_reduce adds
// the blocks.  The columns (snapshots) go in tiles of 16, so a row of J is read once
// per tile.  Per column the 8 rows of a wavefront are added with their signs (the
// same on every lane: factors +-1 in scalar registers), then the sum takes the
// signs of the lane's columns: about one fused multiply-add per coupling and
// snapshot.  grid = (blocks of 32 rows, samples).
__global__ void __launch_bounds__(kDirect) skg_bond_kernel(const SkSample* __restrict__ samples,
                                                           const SkChain* __restrict__ chains, int kd, int nrb,
                                                           int ncol_cap, double* __restrict__ part)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t skg_bits[];   // [kCols][np / 32]
    __shared__ double sums[kDirect / 64][kCols];
    const SkSample* sm = (const SkSample*)(gl(samples) + blockIdx.y);
    const int32_t n = sm->n, np = skg_pitch(n), nw = np >> 5, wn = (n + 31) >> 5;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if ((int32_t)blockIdx.x * kRowsBlk >= n) return;
    const int32_t i0 = (int32_t)blockIdx.x * kRowsBlk + wave * kRows;   // (8 rows of one word of bits)
    const SG_G float* J = gl(sm->Jf) + 4 * lane;
    const int32_t ncol = sm->nch * kd;
    for (int32_t c0 = 0; c0 < ncol; c0 += kCols) {
        __syncthreads();
        for (int32_t w = threadIdx.x; w < kCols * nw; w += kDirect) {
            const int32_t c = w / nw, q = w - c * nw, col = c0 + c, cr = col / kd;
            const SkChain* ch = (const SkChain*)(gl(chains) + sm->chain0 + min(cr, sm->nch - 1));
            skg_bits[w] = col < ncol && q < wn ? gl(ch->snap)[(int64_t)(col - cr * kd) * wn + q] : 0u;
        }
        __syncthreads();
        // bit r: spin i0 + r (rows past n are left out below)
        uint32_t rs[kCols];
#pragma unroll
        for (int c = 0; c < kCols; ++c)
            rs[c] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(skg_bits[c * nw + min(i0 >> 5, nw - 1)] >> (i0 & 31)));
        double acc[kCols];
#pragma unroll
        for (int c = 0; c < kCols; ++c) acc[c] = 0.0;
        for (int32_t q = 0; q < np; q += 256) {
            double x[kRows][4];
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                v4f v = v4f{0.f, 0.f, 0.f, 0.f};
                if (i0 + r < n) v = *(const SG_G v4f*)(J + (int64_t)(i0 + r) * np + q);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[r][e] = (double)v[e];
            }
#pragma unroll
            for (int c = 0; c < kCols; ++c) {
                if (c0 + c >= ncol) break;
                const uint32_t nib = skg_bits[c * nw + (q >> 5) + (lane >> 3)] >> (4 * (lane & 7));
                double t[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    const double s = __hiloint2double((int)(((rs[c] << (31 - r)) & 0x80000000u) | 0x3ff00000u), 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) t[e] = fma(s, x[r][e], t[e]);
                }
                acc[c] += (flip_sign(t[0], nib << 31) + flip_sign(t[1], (nib << 30) & 0x80000000u)) +
                          (flip_sign(t[2], (nib << 29) & 0x80000000u) + flip_sign(t[3], (nib << 28) & 0x80000000u));
            }
        }
        const double v = wave_sum16(acc);
        if ((lane & 3) == 0) sums[wave][sum_index(lane)] = v;
        __syncthreads();
        if (threadIdx.x < kCols && c0 + (int32_t)threadIdx.x < ncol) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < kDirect / 64; ++w) t += sums[w][threadIdx.x];
            part[((int64_t)blockIdx.y * ncol_cap + c0 + threadIdx.x) * nrb + blockIdx.x] = t;
        }
    }
}

// out[chain][k] = (1/2) sum over the row blocks' partial sums, a wavefront each, in
// a fixed order.  grid = (samples, columns)
__global__ void __launch_bounds__(64) skg_bond_reduce(const SkSample* __restrict__ samples, int kd, int nrb,
                                                      int ncol_cap, int k_cap, const double* __restrict__ part,
                                                      double* __restrict__ out)
{
    const SkSample* sm = samples + blockIdx.x;
    const int32_t col = blockIdx.y;
    if (col >= sm->nch * kd) return;
    const int32_t blocks = (sm->n + kRowsBlk - 1) / kRowsBlk;
    const double* p = part + ((int64_t)blockIdx.x * ncol_cap + col) * nrb;
    double v = 0.0;
    for (int32_t i = threadIdx.x; i < blocks; i += 64) v += p[i];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    if (threadIdx.x == 0) out[(int64_t)(sm->chain0 + col / kd) * k_cap + col % kd] = 0.5 * v;
}

}  // namespace

size_t skg_lds_bytes(int32_t n) { return skg_layout(n).total; }

hipError_t skg_diag(const SkSample* samples, int n_samples, const SkChain* chains, int max_n, hipStream_t s)
{
    hipLaunchKernelGGL(skg_diag_kernel, dim3((max_n + 63) / 64, n_samples), dim3(256), 0, s, samples, chains);
    return hipGetLastError();
}

template <int V, int NI>
static hipError_t skg_launch(const SkChain* chains, int n_chains, size_t lds_bytes, int64_t t0, int32_t n_sweeps,
                             int64_t t_max, int* err_flag, hipStream_t s)
{
    // set once (thread-safe initialisation of a local static)
    static const hipError_t attr = hipFuncSetAttribute((const void*)skg_sweep_kernel<V, NI>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return attr;
    skg_sweep_kernel<V, NI><<<dim3(n_chains), dim3(kSkgThreads), lds_bytes, s>>>(chains, t0, n_sweeps, t_max, err_flag);
    return hipGetLastError();
}

// Fields per lane and item: 4 (16-byte loads), fewer while one item per updater
// wavefront covers the chain (N <= 832 and N <= 1664).  Items per wavefront: up to
// 5 at N = 16384.
hipError_t skg_sweep(const SkChain* chains, int n_chains, int max_n, size_t lds_bytes, int64_t t0, int32_t n_sweeps,
                     int64_t t_max, int* err_flag, hipStream_t s)
{
    if (n_chains <= 0 || n_sweeps <= 0) return hipSuccess;
    const int per = (max_n + 256 * kUpd - 1) / (256 * kUpd);
    auto launch = max_n <= 64 * kUpd    ? skg_launch<1, 1>
                  : max_n <= 128 * kUpd ? skg_launch<2, 1>
                  : per <= 1            ? skg_launch<4, 1>
                  : per <= 2            ? skg_launch<4, 2>
                  : per <= 3            ? skg_launch<4, 3>
                  : per <= 4            ? skg_launch<4, 4>
                                        : skg_launch<4, 5>;
    return launch(chains, n_chains, lds_bytes, t0, n_sweeps, t_max, err_flag, s);
}

hipError_t skg_recompute(const SkSample* samples, int n_samples, const SkChain* chains, int max_n, int check,
                         int* err_flag, hipStream_t s)
{
    if (n_samples <= 0) return hipSuccess;
    hipLaunchKernelGGL(skg_recompute_kernel, dim3((max_n + kRowsBlk - 1) / kRowsBlk, n_samples), dim3(kDirect),
                       (size_t)2 * skg_pitch(max_n) / 8, s, samples, chains, check, err_flag);
    return hipGetLastError();
}

int skg_row_blocks(int32_t n) { return (n + kRowsBlk - 1) / kRowsBlk; }

hipError_t skg_bond(const SkSample* samples, int n_samples, const SkChain* chains, int max_n, int max_nch,
                    int k_done, int k_cap, double* part, double* out, hipStream_t s)
{
    if (n_samples <= 0 || k_done <= 0) return hipSuccess;
    const int nrb = skg_row_blocks(max_n), ncol_cap = max_nch * k_cap;
    hipLaunchKernelGGL(skg_bond_kernel, dim3(nrb, n_samples), dim3(kDirect), (size_t)kCols * skg_pitch(max_n) / 8, s,
                       samples, chains, k_done, nrb, ncol_cap, part);
    hipLaunchKernelGGL(skg_bond_reduce, dim3(n_samples, max_nch * k_done), dim3(64), 0, s, samples, k_done, nrb,
                       ncol_cap, k_cap, part, out);
    return hipGetLastError();
}

}  // namespace sg
