// Sherrington-Kirkpatrick Metropolis sweeps on gfx950.
//
// The SK sweep visits i = 0..N-1 in a fixed order (SI, SK section), so a chain
// is sequential.  One workgroup runs one chain, as a pipeline of three roles
// over blocks of 64 consecutive spins (block g of the launch is block b = g mod
// NB of sweep t0 + g / NB).  The couplings are bit-packed by block columns:
// word k of block b holds the signs of J between spin k and the 64 spins of
// block b (bit 1 = -1), so a field's change from the flips of one block is a
// masked popcount of one 64-bit word.  The number of blocks NB is even: spins past
// N are there to fill it and never flip.
//
//  * prep wavefronts (three, ahead of the decider by up to kRing blocks): draw
//    the acceptance uniform r of every position of a block (two Philox streams)
//    and turn it into xmax = max{x : r < thr[x]}, so that a spin with x = s_i
//    H_i flips iff x <= xmax; they also fetch the words of the block's spins
//    for its own columns and for those of the kWin blocks before it.
//  * decider wavefront: lane i owns spin 64 b + i.  It takes the block's fields
//    as published, adds the flips of the blocks since (masked popcounts; for even
//    g the kWin - 1 blocks before, for odd g kWin), and finds the block's flips F as the fixpoint of
//    F = {i : x_i + (change by the flips of F before i) <= xmax_i}.  Lane i's
//    condition depends on lanes before it only, so the fixpoint is unique and is
//    the sequential result; each iteration settles at least one more lane and
//    usually two or three settle all of them (a flip moves x by 2, and few lanes
//    are that close to their bound).  The flips go to a ring buffer.
//  * updater wavefronts (twelve): wavefront w keeps the fields of blocks w, w +
//    12, ... in registers, one field per lane and block, and applies the flips
//    of every pair of blocks to all of them.  The words it needs do not depend on
//    the decisions, so they stream from memory ahead of use, N / 8 bytes per spin
//    and sweep, a spin's words of two blocks in one 16-byte load.  The owners of
//    two coming blocks publish their fields for the decider.
//
// A field is kept as H0 + 2 P - 4 a: P counts the flips applied so far (the
// same for every field) and a the flips that lower it, so that a block costs
// four VALU instructions per field (two three-input logic operations, two
// accumulating popcounts).  A spin's own flips go through the diagonal, which the
// words hold as J_ii = +1: they add 2 s' each, s(now) - s(start) in all, so the
// tracked field is H + s when it starts as H + s.
//
// What bounds it: up to about N = 4096 the decider's own instruction chain (0.42
// to 0.46 us a block: LDS reads, the corrections, 1.5 iterations), above it the
// rate at which one CU takes in words, about 90 GB/s (0.54 us a block at N = 6001,
// 1.42 at 16384).  With 8-byte loads the loads themselves were the bound (N = 4096:
// 0.55 us), and applying flips by reading the coupling rows of the flipped spins,
// as an earlier version did, cost a memory latency per block after each decision
// (1.45 us at N = 512 to 4096, 1.86 at 6001).  Sweeps of 64 x 2 chains, N = 4096:
// 27.2 us, before 97; one chain pair, N = 512: 3.7 us, before 11.4.  A window of 5
// blocks costs the decider more than the slack gives (N = 4096: 31.1 us).  The
// replicas of a sample run on one XCD, so that they share its L2.
//
// Every `period` sweeps the fields are recomputed exactly as H = J S and compared
// with the incremental ones; a mismatch raises the context's error flag.  Bond
// sums B = (1/2) s^T J s of the snapshots are computed at measurement time.
#include <type_traits>

#include "sg_internal.h"
#include "sg_philox.h"
#include "sg_pipe.h"
#include "sg_sk_plan.h"

namespace sg {
namespace {

typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

constexpr int kWin = 3;             // previous blocks whose flips the decider adds itself (odd)
constexpr int kRing = 6;            // blocks the prep wavefronts are ahead at most
constexpr int kHRing = 8;           // published fields of coming blocks
constexpr int kFRing = 64;          // flips of past blocks
constexpr int kEmpty = 4;           // blocks of no flips after the last one
constexpr int kThrCache = 512;      // threshold entries cached in LDS
constexpr int kPrepWaves = 3;
constexpr int kUpdWaves = 12;
constexpr int kSkThreads = 64 * (1 + kPrepWaves + kUpdWaves);
static_assert(64 * kSkLaunchBlocks <= (int64_t)UINT32_MAX, "a launch's accepted flips fit 32 bits");
static_assert(kWin % 2 == 1 && kWin + 3 <= kHRing, "published fields are read before their slots are used again");
// An updater's blocks are at most 2 kUpdWaves - 1 apart, and the decider waits for
// the fields of each, published once the flips kWin + 1 blocks before are applied:
// no updater is further behind than that.
static_assert(kFRing >= kWin + 1 + 2 * kUpdWaves + kEmpty, "flips outlive the slowest updater");
static_assert(kSkOverread >= (size_t)kUpdWaves * 48 * 1024, "slots of the largest variant");
#ifndef SG_SK_PROF
#define SG_SK_PROF 0    // 1: per-role cycle counters, printed by workgroups 0..2 after a launch
#endif
#if SG_SK_PROF
#define SK_CLK(v) const unsigned long long v = clock64()
#define SK_ACC(acc, a, b) (acc) += (b) - (a)
#else
#define SK_CLK(v)
#define SK_ACC(acc, a, b)
#endif

// Previous blocks the decider corrects for in a chain of NB blocks: fewer than NB,
// so that a block never corrects for its own earlier visit (J_ii is not in Jw).
__device__ __forceinline__ int32_t sk_window(int32_t NB) { return min(kWin, NB - 1); }

// LDS byte offsets from the start of the workgroup's dynamic array.
struct SkLds {
    uint32_t h0;      // int32 [64 NB]: field constants H0 (see above)
    uint32_t bits;    // uint64 [NB]: spins, bit 1 = -1
    uint32_t thr;     // uint64 [kThrCache]
    uint32_t xm;      // int32 [kRing][64]: xmax + 1 of a block's spins
    uint32_t row;     // uint64 [kRing][kWin + 1][64]: their words of blocks b, b - 1, ...
    uint32_t hr;      // int32 [kHRing][64]: published fields
    uint32_t flip;    // v4u [kFRing]: flips, spins after the block (two words each)
    uint32_t seqp;    // int32 [kRing]: 1 + block whose xm and row are in the slot
    uint32_t seqh;    // int32 [kHRing]: 1 + block whose fields are in the slot
    uint32_t sync;    // int32 [2]: blocks decided, abort
    uint32_t pr;      // uint4 [kPrepWaves][64]: Philox blocks
    uint32_t total;
};

__host__ __device__ __forceinline__ SkLds sk_layout(int32_t n)
{
    const uint32_t nb = (uint32_t)sk_blocks(n);
    SkLds L;
    uint32_t off = 0;
    auto take = [&](uint32_t bytes) {
        const uint32_t p = off;
        off += (bytes + 15u) & ~15u;
        return p;
    };
    L.h0 = take(nb * 256u);
    L.bits = take(nb * 8u);
    L.thr = take(kThrCache * 8);
    L.xm = take(kRing * 256);
    L.row = take(kRing * (kWin + 1) * 512);
    L.hr = take(kHRing * 256);
    L.flip = take(kFRing * 16);
    L.seqp = take(kRing * 4);
    L.seqh = take(kHRing * 4);
    L.sync = take(8);
    L.pr = take(kPrepWaves * 64 * 16);
    L.total = off;
    return L;
}

__device__ __forceinline__ void wave_sync_sk()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// popcount(v) + acc in the one instruction that does both (left to itself the
// compiler counts from 0 and adds afterwards)
__device__ __forceinline__ uint32_t popc_add(uint32_t v, uint32_t acc)
{
    uint32_t r;
    asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(r) : "v"(v), "v"(acc));
    return r;
}

// ---------------- prep ----------------
__device__ __forceinline__ void sk_prep(const SkChain* ch, const SkLds& L, uint32_t lds, int pw, int64_t t0,
                                        int32_t total)
{
    const int lane = threadIdx.x & 63;
    const int32_t NB = sk_blocks(ch->n), n = ch->n;
    const int32_t cached = min(ch->thr_len, kThrCache), thr_len = ch->thr_len;
    const SG_G uint64_t* __restrict__ gthr = gl(ch->thr);
    const SG_G v2u* __restrict__ Jw = (const SG_G v2u*)gl(ch->Jw);
    const uint32_t thr_o = lds + L.thr;
    auto thr_at = [&](int32_t x) -> unsigned long long {
        return x >= thr_len ? 0ull : x < cached ? *(const SG_L unsigned long long*)(size_t)(thr_o + 8u * (uint32_t)x) : gthr[x];
    };
    v2u tw[kWin + 1];
    auto load_rows = [&](int32_t bq) {
        int32_t c = bq;
#pragma unroll
        for (int d = 0; d <= kWin; ++d) {
            tw[d] = Jw[(((int64_t)(c >> 1) * NB + bq) * 64 + lane) * 2 + (c & 1)];
            c = c == 0 ? NB - 1 : c - 1;
        }
    };
    // block g = (sweep s, index b), advanced by kPrepWaves blocks a turn
    int32_t b = pw, s = 0, slot = pw;
    auto wrap = [&](int32_t& bq, int32_t& sq) {
        while (bq >= NB) {
            bq -= NB;
            ++sq;
        }
    };
    wrap(b, s);
    if (pw < total) load_rows(b);
    for (int32_t g = pw, it = 0; g < total; g += kPrepWaves, ++it) {
        if ((it & 3) == 0) {
            // one pass of the 64 lanes draws both streams' blocks of this
            // wavefront's next four spin blocks: lane 16 j + 8 h + q holds stream
            // h (high / low half-words) of 8-position group q of block g + 3 j
            const int j = lane >> 4;
            int32_t bq = b + kPrepWaves * j, sq = s;
            wrap(bq, sq);
            const uint32_t dom = (lane >> 3) & 1 ? kDomSweepLo : kDomSweepHi;
            const U4 A = philox_stream(ch->seed, (uint32_t)(bq * 8 + (lane & 7)), (uint32_t)(t0 + sq), dom, ch->rep,
                                       ch->inst);
            wave_sync_sk();
            *(SG_L v4u*)(size_t)(lds + L.pr + (uint32_t)(pw * 64 + lane) * 16u) = v4u{A.x, A.y, A.z, A.w};
            wave_sync_sk();
        }
        const uint32_t po = lds + L.pr + (uint32_t)(pw * 64 + (it & 3) * 16 + (lane >> 3)) * 16u + (uint32_t)(lane & 7) * 2u;
        const uint32_t r = ((uint32_t) * (const SG_L uint16_t*)(size_t)po << 16) |
                           (uint32_t) * (const SG_L uint16_t*)(size_t)(po + 128u);
        // starting guess from the logarithm, then exact fix-up on the table
        int32_t x0;
        const float slope = ch->xslope;
        if (slope <= 0.0f) {
            x0 = thr_len - 1;
        } else {
            const float lv = 22.18070977791825f - __logf((float)r + 1.0f);
            const float xf = lv / slope;
            x0 = xf >= (float)(thr_len - 1) ? thr_len - 1 : (xf <= 0.0f ? 0 : (int32_t)xf);
        }
        // (entries cached in LDS first; a long table's tail is read from
        // HBM on a path of its own, so that the common path holds no
        // wait for this wavefront's outstanding loads)
        if (x0 < cached) {
            auto thr_c = [&](int32_t x) { return *(const SG_L unsigned long long*)(size_t)(thr_o + 8u * (uint32_t)x); };
            while (x0 > 0 && !((unsigned long long)r < thr_c(x0))) --x0;
            while (x0 + 1 < cached && (unsigned long long)r < thr_c(x0 + 1)) ++x0;
        }
        if (x0 + 1 >= cached && cached < thr_len) {
            while (x0 > 0 && !((unsigned long long)r < thr_at(x0))) --x0;
            while (x0 + 1 < thr_len && (unsigned long long)r < thr_at(x0 + 1)) ++x0;
        }
        // a lane past the last spin never flips
        if ((b << 6) + lane >= n) x0 = -(1 << 29);
        if (g >= kRing) {
            int spins = 0;
            while (__builtin_amdgcn_readfirstlane(lds_get<int32_t>(lds + L.sync)) < g - kRing + 1) {
                if (wait_giveup(lds + L.sync, spins)) break;
                __builtin_amdgcn_s_sleep(1);
            }
        }
        // (one more: the tracked field is H + s, so s times it is x + 1)
        lds_put<int32_t>(lds + L.xm + (uint32_t)(slot * 64 + lane) * 4u, x0 + 1);
#pragma unroll
        for (int d = 0; d <= kWin; ++d)
            lds_put<v2u>(lds + L.row + (uint32_t)((slot * (kWin + 1) + d) * 64 + lane) * 8u, tw[d]);
        if (lane == 0) lds_put<int32_t>(lds + L.seqp + 4u * (uint32_t)slot, g + 1);
        slot += kPrepWaves;
        if (slot >= kRing) slot -= kRing;
        b += kPrepWaves;
        wrap(b, s);
        if (g + kPrepWaves < total) load_rows(b);
    }
}

// ---------------- decider ----------------
struct SkIn {
    int32_t xm, h, sp, sh;
    v2u row[kWin + 1];
    v2u sb;
};

__device__ __forceinline__ void sk_decide(const SkChain* ch, const SkLds& L, uint32_t lds, int64_t t0, int32_t total,
                                          int64_t t_max)
{
    // the sequential critical path: issue ahead of the wavefronts that share
    // its SIMD
    __builtin_amdgcn_s_setprio(3);
    const int lane = threadIdx.x & 63;
    const int32_t NB = sk_blocks(ch->n), wn = ch->words_n;
    const int32_t DW = sk_window(NB);
    const unsigned long long lt = (1ull << lane) - 1ull;   // lanes before this one
    const uint32_t ltl = (uint32_t)lt, lth = (uint32_t)(lt >> 32);
    uint32_t acc = 0;   // (kSkLaunchBlocks)
    // flips and new spins of the last kWin blocks (d = 0: the block before)
    unsigned long long pF[kWin], pN[kWin];
#pragma unroll
    for (int d = 0; d < kWin; ++d) pF[d] = pN[d] = 0ull;
#if SG_SK_PROF
    unsigned long long tp[4] = {0, 0, 0, 0};   // waiting for inputs, corrections, iterations, their number
#endif
    auto fetch = [&](SkIn& in, int32_t slot, int32_t hslot, int32_t b) __attribute__((always_inline)) {
        in.sp = lds_get<int32_t>(lds + L.seqp + 4u * (uint32_t)slot);
        in.sh = lds_get<int32_t>(lds + L.seqh + 4u * (uint32_t)hslot);
        in.h = lds_get<int32_t>(lds + L.hr + (uint32_t)(hslot * 64 + lane) * 4u);
        in.xm = lds_get<int32_t>(lds + L.xm + (uint32_t)(slot * 64 + lane) * 4u);
#pragma unroll
        for (int d = 0; d <= kWin; ++d)
            in.row[d] = lds_get<v2u>(lds + L.row + (uint32_t)((slot * (kWin + 1) + d) * 64 + lane) * 8u);
        in.sb = lds_get<v2u>(lds + L.bits + 8u * (uint32_t)b);
    };
    int32_t g = 0, b = 0, s = 0, slot = 0;
    SkIn A, B;
    fetch(A, 0, 0, 0);
    // one block: `in` holds (at least an attempt at) its inputs, `nx` gets the next block's
    auto step = [&](SkIn& in, SkIn& nx, auto odd) __attribute__((always_inline)) {
        SK_CLK(c0);
        int spins = 0;
        while (__builtin_amdgcn_readfirstlane((in.sp ^ (g + 1)) | (in.sh ^ (g + 1))) != 0) {
            if (wait_giveup(lds + L.sync, spins)) break;
            fetch(in, slot, g & (kHRing - 1), b);
        }
        SK_CLK(c1);
        SK_ACC(tp[0], c0, c1);
        const unsigned long long SB = ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)in.sb.y) << 32) |
                                      (uint32_t)__builtin_amdgcn_readfirstlane((int)in.sb.x);
        const int32_t nslot = slot + 1 == kRing ? 0 : slot + 1, nb = b + 1 == NB ? 0 : b + 1;
        fetch(nx, nslot, (g + 1) & (kHRing - 1), nb);
        // the flips of the blocks since the fields were published
        uint32_t low = 0;
        int32_t pc = 0;
#pragma unroll
        for (int d = odd ? kWin : kWin - 1; d >= 1; --d) {
            low = popc_add((in.row[d].x ^ (uint32_t)pN[d - 1]) & (uint32_t)pF[d - 1], low);
            low = popc_add((in.row[d].y ^ (uint32_t)(pN[d - 1] >> 32)) & (uint32_t)(pF[d - 1] >> 32), low);
            pc += __popcll(pF[d - 1]);
        }
        const int32_t h = in.h + 2 * pc - 4 * (int32_t)low;
        // x = s h; a flip of lane j < lane raises it by 2 where spins and
        // coupling XOR to 1, else lowers it by 2: lane flips iff
        // 2 (2 up - all) <= xmax - x, up and all counting flips before it
        const int32_t neg = __builtin_amdgcn_inverse_ballot_w64(SB) ? -1 : 0;
        const int32_t m2 = (in.xm - ((h ^ neg) - neg)) >> 1;
        const uint32_t ql = ((uint32_t)SB ^ in.row[0].x ^ (uint32_t)neg) & ltl;
        const uint32_t qh = ((uint32_t)(SB >> 32) ^ in.row[0].y ^ (uint32_t)neg) & lth;
        SK_CLK(c2);
        SK_ACC(tp[1], c1, c2);
        unsigned long long F = __builtin_amdgcn_ballot_w64(m2 >= 0), Fo;
        do {
            Fo = F;
            const uint32_t up = popc_add((uint32_t)(F >> 32) & qh, popc_add((uint32_t)F & ql, 0u));
            const int32_t lim = (int32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(F >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)F, (uint32_t)m2));
            F = __builtin_amdgcn_ballot_w64((int32_t)(2u * up) <= lim);
#if SG_SK_PROF
            ++tp[3];
#endif
        } while (F != Fo);
        SK_CLK(c3);
        SK_ACC(tp[2], c2, c3);
        const unsigned long long SN = SB ^ F;
        if (lane == 0) {
            lds_put<v4u>(lds + L.flip + 16u * ((uint32_t)g & (kFRing - 1)),
                         v4u{(uint32_t)F, (uint32_t)(F >> 32), (uint32_t)SN, (uint32_t)(SN >> 32)});
            lds_put<v2u>(lds + L.bits + 8u * (uint32_t)b, v2u{(uint32_t)SN, (uint32_t)(SN >> 32)});
            lds_put<int32_t>(lds + L.sync, g + 1);
        }
        acc += (uint32_t)__popcll(F);
#pragma unroll
        for (int d = kWin - 1; d > 0; --d) {
            pF[d] = d < (odd ? DW - 1 : DW) ? pF[d - 1] : 0ull;
            pN[d] = pN[d - 1];
        }
        pF[0] = !odd || DW > 1 ? F : 0ull;
        pN[0] = SN;
        ++g;
        slot = nslot;
        b = nb;
        if (b == 0) {
            ++s;
            const int64_t tn = t0 + s;
            if (tn <= t_max && (tn & (tn - 1)) == 0) {
                const int k = 1 + (63 - __clzll((unsigned long long)tn));
                for (int32_t w = lane; w < wn; w += 64)
                    gl(ch->snap)[(int64_t)k * wn + w] = lds_get<uint32_t>(lds + L.bits + 4u * (uint32_t)w);
            }
        }
    };
    while (g < total) {   // (total is even)
        step(A, B, std::false_type{});
        step(B, A, std::true_type{});
    }
    if (lane == 0) {
        for (int e = 0; e < kEmpty; ++e)
            lds_put<v4u>(lds + L.flip + 16u * ((uint32_t)(total + e) & (kFRing - 1)), v4u{0u, 0u, 0u, 0u});
        lds_put<int32_t>(lds + L.sync, total + kEmpty);
    }
    for (int32_t w = lane; w < wn; w += 64) gl(ch->state)[w] = lds_get<uint32_t>(lds + L.bits + 4u * (uint32_t)w);
    if (lane == 0 && acc) atomicAdd(ch->accepted, (unsigned long long)acc);
#if SG_SK_PROF
    if (lane == 0 && blockIdx.x < 3)
        printf("[sk-prof] wg %d decider blocks %d cycles: wait %llu correct %llu iterate %llu; iterations %llu\n",
               (int)blockIdx.x, total, tp[0], tp[1], tp[2], tp[3]);
#endif
}

// ---------------- updaters ----------------
// Wavefront uw holds the fields of blocks uw + kUpdWaves j, j < NG GS, and takes
// them in NG groups of GS; the words of the next D groups are in flight.  (For up
// to 8 fields per lane a group is the whole pair of blocks and D pairs are in
// flight; for more, the groups of one pair take turns in D buffers.)  Slots past
// the last block read the memory after the pair's words (past the last pair, up
// to kSkOverread bytes of the context's memory); what they hold is not used.
template <int NG, int GS, int D>
__device__ __forceinline__ void sk_update(const SkChain* ch, const SkLds& L, uint32_t lds, int uw, int32_t total)
{
    static_assert(NG == 1 || NG % D == 0, "buffers line up with the groups");
    static_assert(NG > 1 || 2 * (D - 1) <= kEmpty, "a last round of D pairs is filled up");
    const int lane = threadIdx.x & 63;
    const int32_t n = ch->n, NB = sk_blocks(n);
    const int32_t ahead = sk_window(NB) + 1;   // fields published after pair (k, k + 1): blocks k + ahead and the next
    if (uw >= NB) return;
    // words of the pair loaded next (index lb)
    const uint64_t Jw = (uint64_t)ch->Jw + (uint64_t)uw * 1024;
    uint64_t src = Jw;
    int32_t lb = 0;
    uint32_t a[NG * GS];
#pragma unroll
    for (int j = 0; j < NG * GS; ++j) a[j] = 0u;
    uint32_t pcs = 0;
    v4u buf[D][GS];
    auto load_next = [&](v4u* dst, int grp) __attribute__((always_inline)) {
        // (scalar bases and one lane offset, made opaque here so that the loads
        // take them as they are: no address arithmetic per lane)
        uint64_t base = src + (uint64_t)(grp * GS * kUpdWaves * 1024);
        uint32_t lofs = 16u * (uint32_t)lane;
        asm("" : "+s"(base), "+v"(lofs));
#pragma unroll
        for (int i = 0; i < GS; ++i)
            dst[i] = *(const SG_G v4u*)((const SG_G char*)(base + (uint64_t)(i * kUpdWaves * 1024)) + lofs);
        __builtin_amdgcn_sched_barrier(0);   // (in order: a wait counts the loads after the ones it waits for)
        if (grp == NG - 1) {
            src += (size_t)NB * 1024;
            if (++lb == NB / 2) {
                lb = 0;
                src = Jw;
            }
        }
    };
    // first block of the pair being applied: k of the launch; block to publish
    // after it: index pb (owner pm, slot pj)
    int32_t k = 0;
    int32_t pb = ahead % NB, pm = pb % kUpdWaves, pj = pb / kUpdWaves;
    auto next = [&](int32_t& x, int32_t& m, int32_t& j) __attribute__((always_inline)) {
        ++x;
        ++m;
        if (m == kUpdWaves) {
            m = 0;
            ++j;
        }
        if (x == NB) x = m = j = 0;
    };
#pragma unroll
    for (int q = 0; q < D; ++q) load_next(buf[q], q % NG);
#if SG_SK_PROF
    unsigned long long tu[2] = {0, 0};   // cycles waiting for decided blocks
#endif
    // flips of the pair's blocks (x, y) and spins after them (z, w), the same
    // in every lane
    v4u f0, f1;
    auto take = [&]() __attribute__((always_inline)) {
        SK_CLK(u0);
        int spins = 0;
        const uint32_t fo = lds + L.flip + 16u * ((uint32_t)k & (kFRing - 1));
#pragma unroll 1
        for (;;) {
            const int32_t dec = lds_get<int32_t>(lds + L.sync);
            f0 = lds_get<v4u>(fo);
            f1 = lds_get<v4u>(fo + 16u);
            if (__builtin_amdgcn_readfirstlane(dec) > k + 1) break;
            if (wait_giveup(lds + L.sync, spins)) break;
            __builtin_amdgcn_s_sleep(1);
        }
        SK_CLK(u1);
        SK_ACC(tu[0], u0, u1);
    };
    auto apply = [&](const v4u* w, int grp) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < GS; ++i) {
            uint32_t c = a[grp * GS + i];
            c = popc_add(f0.x & (w[i].x ^ f0.z), c);
            c = popc_add(f0.y & (w[i].y ^ f0.w), c);
            c = popc_add(f1.x & (w[i].z ^ f1.z), c);
            a[grp * GS + i] = popc_add(f1.y & (w[i].w ^ f1.w), c);
        }
    };
    auto field = [&](int32_t blk, uint32_t cnt) {
        return lds_get<int32_t>(lds + L.h0 + (uint32_t)(blk * 64 + lane) * 4u) + (int32_t)(2u * pcs) - (int32_t)(4u * cnt);
    };
    // after the last group of the pair
    auto finish = [&]() __attribute__((always_inline)) {
        pcs = popc_add(f0.x, popc_add(f0.y, popc_add(f1.x, popc_add(f1.y, pcs))));
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int32_t g = k + ahead + h;
            if (pm == uw && g < total) {
                uint32_t c = a[0];
#pragma unroll
                for (int j = 1; j < NG * GS; ++j) {
                    c = pj == j ? a[j] : c;
                    asm("" : "+v"(c));   // (selects: a chain seen as an indexed read would go through scratch memory)
                }
                lds_put<int32_t>(lds + L.hr + (uint32_t)((g & (kHRing - 1)) * 64 + lane) * 4u, field(pb, c));
                if (lane == 0) lds_put<int32_t>(lds + L.seqh + 4u * (uint32_t)(g & (kHRing - 1)), g + 1);
            }
            next(pb, pm, pj);
        }
        k += 2;
    };
    // (whole rounds of D pairs: a way out of the middle of a round would join
    // the loop's end with other loads in flight, and the waits for the oldest words
    // would become waits for all; the decider ends with kEmpty blocks of no flips)
    while (k < total) {
        if (NG == 1) {
#pragma unroll
            for (int q = 0; q < D; ++q) {
                take();
                apply(buf[q], 0);
                finish();
                load_next(buf[q], 0);
            }
        } else {
            take();
#pragma unroll
            for (int grp = 0; grp < NG; ++grp) {
                apply(buf[grp % D], grp);
                load_next(buf[grp % D], (grp + D) % NG);
            }
            finish();
        }
    }
#pragma unroll
    for (int j = 0; j < NG * GS; ++j) {
        const int32_t blk = uw + kUpdWaves * j, i = blk * 64 + lane;
        if (i < n) {
            const uint32_t w = lds_get<uint32_t>(lds + L.bits + 4u * (uint32_t)(i >> 5));
            gl(ch->H)[i] = field(blk, a[j]) - 1 + 2 * (int32_t)((w >> (lane & 31)) & 1u);
        }
    }
#if SG_SK_PROF
    if (lane == 0 && blockIdx.x < 3)
        printf("[sk-prof] wg %d updater %d cycles waiting %llu\n", (int)blockIdx.x, uw, tu[0]);
#endif
}

template <int NG, int GS, int D>
__global__ void __launch_bounds__(kSkThreads) sk_sweep_kernel(const SkChain* __restrict__ chains, int64_t t0,
                                                              int32_t nsw, int64_t t_max, int* err)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t sk_smem[];
    const SkChain* ch = (const SkChain*)(gl(chains) + chain_of_block(blockIdx.x, gridDim.x));
    const uint32_t lds = (uint32_t)(size_t)(SG_L uint8_t*)sk_smem;
    const int32_t n = ch->n, wn = ch->words_n, NB = sk_blocks(n);
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const SkLds L = sk_layout(n);
    const int32_t total = nsw * NB;   // (bounded by the host)
    const int32_t DW = sk_window(NB);
    const SG_G int32_t* gH = gl(ch->H);
    const SG_G uint32_t* gst = gl(ch->state);
    const SG_G uint64_t* gthr = gl(ch->thr);
    // (the diagonal counts as J_ii = +1 in the sweep: tracked fields are H + s)
    for (int32_t i = tid; i < 64 * NB; i += nthr) {
        const int32_t h = i < n ? gH[i] + 1 - 2 * (int32_t)((gst[i >> 5] >> (i & 31)) & 1u) : 0;
        lds_put<int32_t>(lds + L.h0 + 4u * (uint32_t)i, h);
        // the fields of the first blocks, which no flip precedes by more than
        // the window
        if (i < 64 * (DW + 1)) lds_put<int32_t>(lds + L.hr + 4u * (uint32_t)i, h);
    }
    for (int32_t w = tid; w < 2 * NB; w += nthr) lds_put<uint32_t>(lds + L.bits + 4u * (uint32_t)w, w < wn ? gst[w] : 0u);
    for (int32_t x = tid; x < min(ch->thr_len, kThrCache); x += nthr)
        lds_put<uint64_t>(lds + L.thr + 8u * (uint32_t)x, gthr[x]);
    if (tid < kRing) lds_put<int32_t>(lds + L.seqp + 4u * (uint32_t)tid, 0);
    if (tid < kHRing) lds_put<int32_t>(lds + L.seqh + 4u * (uint32_t)tid, tid <= DW ? tid + 1 : 0);
    if (tid < 2) lds_put<int32_t>(lds + L.sync + 4u * (uint32_t)tid, 0);
    __syncthreads();
    // Wavefronts go to the four SIMDs in turn: the decider shares its SIMD with
    // the prep wavefronts, the updaters have the other three.
    if (wave == 0)
        sk_decide(ch, L, lds, t0, total, t_max);
    else if ((wave & 3) == 0)
        sk_prep(ch, L, lds, (wave >> 2) - 1, t0, total);
    else
        sk_update<NG, GS, D>(ch, L, lds, wave - 1 - (wave >> 2), total);
    __syncthreads();
    if (tid == 0 && lds_get<int32_t>(lds + L.sync + 4)) atomicOr(err, 2);
}

// Initial configuration and the t = 0 snapshot of every chain.
__global__ void sk_init_kernel(const SkChain* __restrict__ chains)
{
    const SkChain* ch = chains + blockIdx.x;
    const int32_t n = ch->n, wn = ch->words_n;
    for (int32_t w = threadIdx.x; w < wn; w += blockDim.x) {
        uint32_t bits;
        if (ch->init_mode == 0) {
            const U4 o = philox_stream(ch->seed, (uint32_t)(w >> 2), 0u, kDomInit, ch->rep, ch->inst);
            bits = word_of(o, (uint32_t)(w & 3));
        } else if (ch->init_mode == 1) {
            bits = 0;
        } else {
            bits = ch->given[w];
        }
        const int32_t pe = n - 32 * w;
        if (pe < 32) bits &= (1u << pe) - 1u;
        ch->state[w] = bits;
        ch->snap[w] = bits;
    }
}

// ---------------- exact sums ----------------
// H = J S and the bond sums s^T J s are +-1 contractions.  They run on the packed
// words: 32 products are one XOR and one accumulating popcount of a lane, on an
// eighth of the bytes that int8 couplings take, and the words are there for the
// sweep already.  64 x 2 chains of N = 4096: fields 38 us (3.5 TB/s of words) and 12
// snapshots a chain 179 us, against 263 and 460 us by int8 MFMA on int8 couplings,
// which read N^2 bytes per sample and column tile and expanded every spin; 4 x 2
// chains of N = 6001, whose int8 rows were not 16-byte aligned: 13.5 and 36 us
// against 377 and 446.
// Four words of spins of pair p (zeros past the last word).
__device__ __forceinline__ v4u sk_spins(const SG_G uint32_t* st, int32_t p, int32_t wn)
{
    if (4 * p + 3 < wn) {
        const SG_G uint32_t* q = st + 4 * p;
        return v4u{q[0], q[1], q[2], q[3]};
    }
    return v4u{4 * p < wn ? st[4 * p] : 0u, 4 * p + 1 < wn ? st[4 * p + 1] : 0u, 4 * p + 2 < wn ? st[4 * p + 2] : 0u, 0u};
}

__device__ __forceinline__ uint32_t sk_differ(const v4u& w, const v4u& s, uint32_t acc)
{
    return popc_add(w.x ^ s.x, popc_add(w.y ^ s.y, popc_add(w.z ^ s.z, popc_add(w.w ^ s.w, acc))));
}

// Words of spin k for the pairs p0 + wave, p0 + wave + 4, ... (8 of them, fewer at
// the end): bits that differ from a column's spins are products -1.
constexpr int kDotPairs = 8;   // pairs per wavefront and pass: 4 wavefronts cover 4096 columns

struct SkWords {
    v4u w[kDotPairs];
    int32_t np;   // (wave-uniform)
};

__device__ __forceinline__ void sk_words(SkWords& W, const SG_G v4u* Jw, int32_t NB, int32_t k, int32_t p0, int wave)
{
    W.np = max(0, min(kDotPairs, (NB / 2 - p0 - wave + 3) / 4));
#pragma unroll
    for (int i = 0; i < kDotPairs; ++i)
        if (i < W.np) W.w[i] = Jw[(int64_t)(p0 + wave + 4 * i) * 64 * NB + k];
}

// Exact fields for all chains of one sample, compared with the incremental ones
// when `check`.  Block = 64 spins, its four wavefronts share the columns;
// grid = (blocks of 64 spins, samples).
template <int C>
__global__ void __launch_bounds__(256) sk_recompute_kernel(const SkSample* __restrict__ samples,
                                                           const SkChain* __restrict__ chains,
                                                           int check, int* err)
{
    __shared__ uint32_t part[4][C][64];
    const SkSample* sm = (const SkSample*)(gl(samples) + blockIdx.y);
    const int32_t n = sm->n, nch = sm->nch, NB = sk_blocks(n), wn = (n + 31) >> 5;
    if ((int32_t)blockIdx.x >= NB) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const SkChain* ch = (const SkChain*)(gl(chains) + sm->chain0);
    uint32_t cnt[C];
#pragma unroll
    for (int c = 0; c < C; ++c) cnt[c] = 0u;
    for (int32_t p0 = 0; p0 < NB / 2; p0 += 4 * kDotPairs) {
        SkWords W;
        sk_words(W, (const SG_G v4u*)gl(sm->Jw), NB, (int32_t)blockIdx.x * 64 + lane, p0, wave);
#pragma unroll
        for (int i = 0; i < kDotPairs; ++i) {
            if (i >= W.np) break;
#pragma unroll
            for (int c = 0; c < C; ++c)
                if (c < nch) cnt[c] = sk_differ(W.w[i], sk_spins(gl(ch[c].state), p0 + wave + 4 * i, wn), cnt[c]);
        }
    }
#pragma unroll
    for (int c = 0; c < C; ++c) part[wave][c][lane] = cnt[c];
    __syncthreads();
    const int32_t i = (int32_t)blockIdx.x * 64 + lane;
    for (int c = wave; c < nch; c += 4) {
        if (i >= n) break;
        const uint32_t d = part[0][c][lane] + part[1][c][lane] + part[2][c][lane] + part[3][c][lane];
        // (the diagonal counts as +1 in the words: s_i taken off)
        const int32_t si = 1 - 2 * (int32_t)((gl(ch[c].state)[i >> 5] >> (i & 31)) & 1u);
        const int32_t h = n - 2 * (int32_t)d - si;
        SG_G int32_t* H = gl(ch[c].H);
        if (check && H[i] != h) atomicOr(err, 1);
        H[i] = h;
    }
}

// Bond sums of the snapshots: adds 2 B = sum_i s_i (J s)_i of every column (chain
// r, snapshot k) of one sample into out[chain][k].  A block takes the products of
// 64 spins with up to 4096 others, whose words it holds in registers while the
// columns pass in tiles of 8; grid = (blocks of 64 spins, passes, samples).
__global__ void __launch_bounds__(256) sk_bond_kernel(const SkSample* __restrict__ samples,
                                                      const SkChain* __restrict__ chains, int kd,
                                                      int k_cap, long long* __restrict__ out)
{
    constexpr int CT = 8;
    __shared__ int32_t part[CT][256];
    const SkSample* sm = (const SkSample*)(gl(samples) + blockIdx.z);
    const int32_t n = sm->n, NB = sk_blocks(n), wn = (n + 31) >> 5, ncol = sm->nch * kd;
    const int32_t p0 = (int32_t)blockIdx.y * 4 * kDotPairs;
    if ((int32_t)blockIdx.x >= NB || p0 >= NB / 2) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int32_t i = (int32_t)blockIdx.x * 64 + lane;
    SkWords W;
    sk_words(W, (const SG_G v4u*)gl(sm->Jw), NB, i, p0, wave);
    const SkChain* ch = (const SkChain*)(gl(chains) + sm->chain0);
    for (int32_t c0 = 0; c0 < ncol; c0 += CT) {
        uint32_t cnt[CT];
        const SG_G uint32_t* col[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int32_t q = min(c0 + c, ncol - 1), cr = q / kd;
            col[c] = gl(ch[cr].snap) + (int64_t)(q - cr * kd) * wn;
            cnt[c] = 0u;
        }
#pragma unroll
        for (int w = 0; w < kDotPairs; ++w) {
            if (w >= W.np) break;
#pragma unroll
            for (int c = 0; c < CT; ++c) cnt[c] = sk_differ(W.w[w], sk_spins(col[c], p0 + wave + 4 * w, wn), cnt[c]);
        }
        // s_i (products) of this wavefront's columns; the first pass's first
        // wavefront adds s_i (n - s_i), the count of products less the diagonal
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const int32_t si = i < n ? 1 - 2 * (int32_t)((col[c][i >> 5] >> (i & 31)) & 1u) : 0;
            const int32_t base = p0 == 0 && wave == 0 ? n - si : 0;
            part[c][threadIdx.x] = si * (base - 2 * (int32_t)cnt[c]);
        }
        __syncthreads();
        // 32 threads per column
        const int c = threadIdx.x >> 5, t = threadIdx.x & 31;
        int32_t v = 0;
#pragma unroll
        for (int q = 0; q < 8; ++q) v += part[c][t + 32 * q];
#pragma unroll
        for (int o = 16; o >= 1; o >>= 1) v += __shfl_xor(v, o);
        if (t == 0 && c0 + c < ncol && v != 0) {
            const int32_t q = c0 + c, cr = q / kd;
            atomicAdd((unsigned long long*)&out[(int64_t)(sm->chain0 + cr) * k_cap + (q - cr * kd)],
                      (unsigned long long)(long long)v);
        }
        __syncthreads();
    }
}

}  // namespace

size_t sk_lds_bytes(int32_t n) { return sk_layout(n).total; }

hipError_t sk_init(const SkChain* chains, int n_chains, int threads, hipStream_t s)
{
    if (n_chains <= 0) return hipSuccess;
    hipLaunchKernelGGL(sk_init_kernel, dim3(n_chains), dim3(threads), 0, s, chains);
    return hipGetLastError();
}

hipError_t sk_recompute(const SkSample* samples, int n_samples, const SkChain* chains, int max_n, int max_nch,
                        int check, int* err_flag, hipStream_t s)
{
    if (n_samples <= 0) return hipSuccess;
    auto k = max_nch <= 1   ? sk_recompute_kernel<1>
             : max_nch <= 2 ? sk_recompute_kernel<2>
             : max_nch <= 4 ? sk_recompute_kernel<4>
                            : sk_recompute_kernel<8>;
    hipLaunchKernelGGL(k, dim3(sk_blocks(max_n), n_samples), dim3(256), 0, s, samples, chains, check, err_flag);
    return hipGetLastError();
}

hipError_t sk_bond(const SkSample* samples, int n_samples, const SkChain* chains, int max_n, int k_done, int k_cap,
                   long long* out, hipStream_t s)
{
    if (n_samples <= 0 || k_done <= 0) return hipSuccess;
    const int nb = sk_blocks(max_n), pass = 2 * 4 * kDotPairs;
    dim3 grid(nb, (nb + pass - 1) / pass, n_samples);
    hipLaunchKernelGGL(sk_bond_kernel, grid, dim3(256), 0, s, samples, chains, k_done, k_cap, out);
    return hipGetLastError();
}

// Fields per lane of an updater: ceil(blocks / 12), held in NG groups of GS.
template <int NG, int GS, int D>
static hipError_t sk_launch(const SkChain* chains, int n_chains, size_t lds_bytes, int64_t t0, int32_t n_sweeps,
                            int64_t t_max, int* err_flag, hipStream_t s)
{
    // set once (thread-safe initialisation of a local static)
    static const hipError_t attr = hipFuncSetAttribute((const void*)sk_sweep_kernel<NG, GS, D>,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return attr;
    sk_sweep_kernel<NG, GS, D><<<dim3(n_chains), dim3(kSkThreads), lds_bytes, s>>>(chains, t0, n_sweeps, t_max, err_flag);
    return hipGetLastError();
}

hipError_t sk_sweep(const SkChain* chains, int n_chains, int max_n, size_t lds_bytes, int64_t t0,
                    int32_t n_sweeps, int64_t t_max, int* err_flag, hipStream_t s)
{
    if (n_chains <= 0 || n_sweeps <= 0) return hipSuccess;
    const int per = (sk_blocks(max_n) + kUpdWaves - 1) / kUpdWaves;
    auto launch = per <= 1    ? sk_launch<1, 1, 3>
                  : per <= 2  ? sk_launch<1, 2, 3>
                  : per <= 3  ? sk_launch<1, 3, 3>
                  : per <= 4  ? sk_launch<1, 4, 3>
                  : per <= 5  ? sk_launch<1, 5, 3>
                  : per <= 6  ? sk_launch<1, 6, 3>
                  : per <= 7  ? sk_launch<1, 7, 2>
                  : per <= 8  ? sk_launch<1, 8, 2>
                  : per <= 12 ? sk_launch<2, 6, 2>
                  : per <= 16 ? sk_launch<4, 4, 4>
                  : per <= 24 ? sk_launch<6, 4, 2>
                  : per <= 32 ? sk_launch<8, 4, 2>
                              : sk_launch<12, 4, 2>;
    return launch(chains, n_chains, lds_bytes, t0, n_sweeps, t_max, err_flag, s);
}

}  // namespace sg
