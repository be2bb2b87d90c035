// Viana-Bray Metropolis sweeps on gfx950.
//
// One workgroup owns one work unit: a graph stored in sweep order (the
// colour classes of a proper colouring, the paper's bipartite parallel update
// generalised; SI "Simulations of the Bethe Lattice on GPUs") and up to eight
// chains that share it.  The chains' spins stay in LDS for the whole launch in
// the sliced packing of VbLayout (one 32-bit word = P = 32 / rpad consecutive
// positions of every chain, chain c in its own P-bit field), so that one LDS
// read of a neighbour's word returns its spin in every chain and the
// unsatisfied-bond counts of all chains advance with one shift, XOR, mask and
// add (4-bit fields while every degree of the chunk is below 16, else two
// sets of 8-bit fields).
//
// A sweep visits colour class 0, 1, ...; inside a class all positions are
// independent (no two are adjacent).  A class is cut into chunks of two aligned
// blocks of 64 positions (one block where the adjacency is resident in LDS, and in some
// split units: split_chunk_blocks), which
// the wavefronts take in turn; lane i of a wavefront updates position i of each
// block for every chain of the unit.  vb_loop says how the wavefronts keep the
// order of the classes and what is in flight when.
//
// Metropolis rule (Methods; SI bipartite-graph section): with x = s_p h_p the
// move is accepted if x <= 0, else iff r < thr[x], thr[x] = floor(2^32
// exp(-2x/T)).  r = (A << 16) | B with A, B half-words of two Philox streams.
// One Philox block serves the eight positions of an aligned group for one
// chain.  A wavefront draws 64 of them per pass (one per lane): those of its next
// B = max(1, 8 / nch) blocks of positions, so with 1, 2 or 4 chains no lane draws
// what nobody uses; they reach the positions' lanes through LDS.  A is compared with the high half of the threshold,
// read from a per-chain table indexed by 64 + x (entries for x <= 0 exceed
// every A); B is computed only when A ties with it (probability 2^-16).
#include <type_traits>

#include "sg_internal.h"
#include "sg_philox.h"

namespace sg {
namespace {

// neighbours of a position kept in registers, adjacency in HBM / in LDS
constexpr int kHbmMax = 8, kLdsMax = 12;
constexpr int kTab = 128;  // threshold table per chain: index 64 + x, -63 <= x <= 63
constexpr int kThc = 32;   // compact threshold table per chain: index 15 - x, -16 <= x <= 15
constexpr int kMaxCls = 64; // colour classes (greedy colouring, degree <= 63)
// LDS byte offsets of the flip-spreading table (256 words) and of the spin
// words: the compact tables come first, so that all three are addressed
// with the instructions' constant offsets
constexpr uint32_t kSprOff = kVbMaxChains * kThc * 4;
constexpr uint32_t kSpOff = kSprOff + 256 * 4;

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Compile-time form of VbLayout for a unit with RPAD chain slots.
template <int RPAD>
struct Sl {
    static constexpr int P = 32 / RPAD;             // positions per word (= field width)
    static constexpr int LP = RPAD == 1 ? 5 : RPAD == 2 ? 4 : RPAD == 4 ? 3 : 2;   // log2 P
    // field bottoms; for RPAD 8 the 4-bit fields
    static constexpr uint32_t M = RPAD == 1 ? 1u : RPAD == 2 ? 0x00010001u : RPAD == 4 ? 0x01010101u : 0x11111111u;
    // byte offset in LDS of the word holding position (en & 0x7fffffff); the
    // sign bit of an adjacency entry is masked off
    static __device__ __forceinline__ uint32_t boff(uint32_t en)
    {
        return (en & (0x7fffffffu & ~(uint32_t)(P - 1))) >> (LP - 2);
    }
};

struct VbLds {
    uint32_t* thc;                // [8][kThc] at LDS offset 0: 15 - x -> thr[x] >> 16; 0x10000 for x <= 0
    uint32_t* spr;                // [256] at kSprOff: bit c of v -> bit 4 c of spr[v]
    uint32_t* sp;                 // spins, VbLayout words, at LDS offset kSpOff
    uint32_t sp_lds;              // the same array as a byte offset in LDS
    uint32_t* cp;                 // (units with cpl) the complemented words
    uint32_t cp_lds;
    uint32_t* thr;                // [8][kTab]: 64 - x -> thr[x] >> 16; 0x10000 for x <= 0
    unsigned long long* accs;     // [8]
    int32_t* flag;                // [4]: split units' abort flag
    int32_t* cls;                 // [kMaxCls + 1] first position of each colour class
    uint32_t* ri;                 // [8][2]: replica, instance of each chain
    uint32_t* wacc;               // [kMaxGrid][8]: window overlap counts of a sweep
    uint4* xch;                   // [waves][64] Philox blocks of a batch of chunks
    int32_t* area;                // resident adjacency: row starts, then entries
};

// Chunks whose Philox blocks one pass of 64 lanes draws.
__host__ __device__ __forceinline__ int32_t vb_batch_chunks(int32_t nch)
{
    return nch <= 8 ? (8 / nch > 0 ? 8 / nch : 1) : 1;
}

__device__ __forceinline__ VbLds vb_carve(uint32_t* smem, uint32_t smem_lds, int32_t sw, int nthr, int32_t nch,
                                          bool cpl)
{
    VbLds L;
    const int32_t swp = (sw + 3) & ~3;
    L.thc = smem;
    L.spr = smem + kSprOff / 4;
    L.sp = smem + kSpOff / 4;
    L.sp_lds = smem_lds + kSpOff;
    L.cp = L.sp + swp;
    L.cp_lds = L.sp_lds + 4u * (uint32_t)swp;
    L.thr = L.sp + (cpl ? 2 * swp : swp);
    L.accs = (unsigned long long*)(L.thr + kVbMaxChains * kTab);
    L.flag = (int32_t*)(L.accs + kVbMaxChains);
    L.cls = L.flag + 4;
    L.ri = (uint32_t*)(L.cls + kMaxCls + 4);
    L.wacc = L.ri + 2 * kVbMaxChains;
    L.xch = (uint4*)(L.wacc + kMaxGrid * kVbMaxChains);
    L.area = (int32_t*)(L.xch + (nthr >> 6) * 64);
    return L;
}

// A value that is the same in every lane, in scalar registers.
__device__ __forceinline__ int64_t uniform64(int64_t v)
{
    return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int32_t)((uint64_t)v >> 32)) << 32) |
                     (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)v));
}

template <class T>
__device__ __forceinline__ T* uniform(T* p)
{
    return (T*)uniform64((int64_t)p);
}

// Class bounds, wave-uniform.
__device__ __forceinline__ int32_t cls_at(const int32_t* cls, int32_t k)
{
    return __builtin_amdgcn_readfirstlane(cls[k]);
}

typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef v4u v4u_dw __attribute__((aligned(4)));

// Adjacency rows and the first NE entries of one chunk of H blocks of 64
// positions, as read (from HBM or LDS).
template <int NE, int H>
struct Stage {
    int32_t r0[H], deg[H];     // row start, degree (as requested: the row's end; 0 in lanes outside the class)
    v4u e[H][NE / 4];
};

// (HBM: one 16-byte load; rows start at any entry)
__device__ __forceinline__ v4u entries4(const SG_G uint32_t* ent, int32_t r0, int d)
{
    const uint32_t o = (uint32_t)r0 * 4u;
    return *(const SG_G v4u_dw*)((const SG_G char*)(ent + d) + o);
}

__device__ __forceinline__ v4u entries4(const uint32_t* ent, int32_t r0, int d)
{
    const uint32_t* p = ent + r0 + d;
    return v4u{p[0], p[1], p[2], p[3]};
}

// The rows of a chunk: requested one chunk ahead, except where every lane has the
// same degree (most chunks: positions are sorted by degree inside a class), whose
// rows follow from the first one.
template <class PR, int NE, int H>
__device__ __forceinline__ void load_rows(PR row, const VbChunk& T, int lane, Stage<NE, H>& st)
{
    if (T.even()) return;
#pragma unroll
    for (int h = 0; h < H; ++h) {
        // (clamped in lanes past the class)
        const uint32_t q = (uint32_t)min(T.base() + 64 * h + lane, T.base() + T.hi() - 1);
        st.r0[h] = row[q];
        st.deg[h] = row[q + 1];
    }
}

__device__ __forceinline__ bool in_class(const VbChunk& T, int lane)
{
    return lane >= T.lo() && lane < T.hi();
}

// The rows of chunk T (in `rows`, if they were requested) as row starts and degrees.
template <int NE, int H>
__device__ __forceinline__ void rows_ready(Stage<NE, H>& st, const Stage<NE, H>& rows, const VbChunk& T, int lane)
{
    if (T.even()) {
#pragma unroll
        for (int h = 0; h < H; ++h) {
            st.r0[h] = (int32_t)T.r0 + (int32_t)((uint32_t)(64 * h + lane) * (uint32_t)T.degree());
            st.deg[h] = T.degree();
        }
    } else {
#pragma unroll
        for (int h = 0; h < H; ++h) {
            st.r0[h] = rows.r0[h];
            st.deg[h] = in_class(T, 64 * h + lane) ? rows.deg[h] - rows.r0[h] : 0;
        }
    }
}

// Loads the entries from the row start whatever the lane's degree (the adjacency
// is followed by kVbEntPad zero entries), four at a time up to the chunk's largest.
template <class PE, int NE, int H>
__device__ __forceinline__ void load_ents(PE ent, Stage<NE, H>& st, int32_t degree)
{
    static_assert(NE <= kVbEntPad, "entry prefetch must stay inside the padded adjacency");
#pragma unroll
    for (int i = 0; i < NE / 4; ++i) {
        if (i == 0 || degree > 4 * i) {
#pragma unroll
            for (int h = 0; h < H; ++h) st.e[h][i] = entries4(ent, st.r0[h], 4 * i);
        }
    }
}

// A lane's random half-words A of a chunk, and the low half-word B that decides a
// tie (drawn when it is needed: probability 2^-16).
template <int RPAD, int H>
struct Draws {
    // (8 slots, two blocks: the first block's stay in LDS, for want of registers)
    static constexpr int R0 = RPAD == 8 && H == 2 ? 1 : 0;
    uint32_t a[H - R0][RPAD];
    const uint16_t* first;
    __device__ __forceinline__ uint32_t half(int h, int c) const
    {
        return R0 && h == 0 ? (uint32_t)first[8 * c] : a[h - R0 < 0 ? 0 : h - R0][c];
    }
};

struct Site {
    const VbUnit* up;
    uint64_t key;
    uint32_t t;
    int32_t q;      // position (of the first block)
    int32_t nch;
};

// Half-word of the lane's position in block h for chain c (not a constant).
__device__ __forceinline__ uint32_t site_half(const Site& S, uint32_t domain, int h, int c)
{
    const uint32_t q = (uint32_t)S.q + 64u * (uint32_t)h;
    return half_word(philox_stream(S.key, q >> 3, S.t, domain, S.up->rep[c], S.up->inst[c]), q & 7u);
}

// Metropolis decisions of one chunk for every chain, from the unsatisfied-bond
// counts: chain c's count is the `width`-bit field of cA (c even or RPAD < 8)
// or cB (c odd, RPAD 8, 8-bit fields) at bit fsh(c).  Makes fl this lane's flips
// in spin-word form (chain c's flip at bit c P).  The counts index the full tables
// (x = deg - 2 cnt at word c kTab + 64 - x).
template <int RPAD, int H>
__device__ __forceinline__ void vb_decide_full(const Site& site, const VbLds& L, const Draws<RPAD, H>& A,
                                               const uint32_t (&cA)[H], const uint32_t (&cB)[H], const int32_t (&deg)[H],
                                               const bool (&act)[H], uint32_t (&fl)[H])
{
    using S = Sl<RPAD>;
    constexpr uint32_t width = RPAD == 8 ? 8u : (uint32_t)S::P;
    // (the counts are selected as values: a selected reference would put
    // cA and cB in private memory when c is not a constant)
    auto count = [&](int h, int c) -> uint32_t {
        const uint32_t a = cA[h], b = cB[h];
        if (RPAD == 1) return a;
        const uint32_t fsh = RPAD == 8 ? 8u * (uint32_t)(c >> 1) : (uint32_t)(c * S::P);
        return __builtin_amdgcn_ubfe(RPAD == 8 && (c & 1) ? b : a, fsh, width);
    };
    // (the address includes the lane's 4 (64 - deg): a single shift-add)
    auto thr_of = [&](int h, int c, uint32_t cnt) -> uint32_t {
        return *(const uint32_t*)((const char*)L.thr + (uint32_t)(64 - deg[h]) * 4u + c * kTab * 4 + (cnt << 3));
    };
    // e = A - thr (|e| < 2^18): a flip iff e < 0, a tie iff e = 0
    uint32_t emin[H];
#pragma unroll
    for (int h = 0; h < H; ++h) {
        fl[h] = 0u;
        emin[h] = 0xFFFFFFFFu;
    }
    auto chain = [&](int c) {
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const uint32_t e = A.half(h, c) - thr_of(h, c, count(h, c));
            fl[h] |= (e >> 31) << (c * S::P);
            emin[h] = min(emin[h], e);
        }
    };
    // a unit with RPAD slots has more than RPAD / 2 chains: those are decided
    // without a test (in one block, so that their LDS reads are issued together)
#pragma unroll
    for (int c = 0; c <= RPAD / 2; ++c) chain(c);
#pragma unroll
    for (int c = RPAD / 2 + 1; c < RPAD; ++c)
        if (c < site.nch) chain(c);
#pragma unroll
    for (int h = 0; h < H; ++h) {
        fl[h] = act[h] ? fl[h] : 0u;
        if (__builtin_amdgcn_ballot_w64(act[h] && emin[h] == 0u) != 0ull) {
            // A equals the high half of the threshold (those lanes did not flip
            // above): decide on the low half (rare: a loop, not unrolled)
            if (act[h] && emin[h] == 0u) {
#pragma unroll 1
                for (int c = 0; c < site.nch; ++c) {
                    const uint32_t cnt = count(h, c);
                    if (site_half(site, kDomSweepHi, h, c) == thr_of(h, c, cnt) &&
                        site_half(site, kDomSweepLo, h, c) < gl(&site.up->thr_lo[c][0])[deg[h] - 2 * (int32_t)cnt])
                        fl[h] |= 1u << (c * S::P);
                }
            }
        }
    }
}

// The same with 8 chain slots and every degree of the chunk below 16 (the
// usual case), in fewer instructions.  The 4-bit counts are spread to bytes
// (even chains in oE, odd chains in oO, chain c at byte c / 2) and each byte
// is turned, for all chains at once, into the byte offset 4 (15 - x) = 60 -
// 4 deg + 8 cnt of the chain's entry in its compact table at LDS offset 0,
// so that one bit-field extract per chain addresses its threshold; e = A - thr
// (|e| < 2^17) decides: a flip iff e < 0, a tie iff e = 0.  The sign bits are
// shifted into a flip vector (bit c: chain c, from the highest chain down),
// which the spreading table turns into spin-word form; ties are detected by the
// running unsigned minimum of e.
template <int H>
__device__ __forceinline__ void vb_decide_compact(const Site& site, const Draws<8, H>& A, const uint32_t (&cA)[H],
                                                  const int32_t (&deg)[H], const bool (&act)[H], uint32_t (&fl)[H])
{
    typedef const __attribute__((address_space(3))) uint32_t lds_u32;
    uint32_t oE[H], oO[H], fv[H], emin[H];
#pragma unroll
    for (int h = 0; h < H; ++h) {
        // (60 - 4 deg) in every byte
        const uint32_t bias = __builtin_amdgcn_perm(0u, (uint32_t)(60 - 4 * deg[h]), 0u);
        oE[h] = ((cA[h] & 0x0F0F0F0Fu) << 3) + bias;          // chain 2k at byte k
        oO[h] = (((cA[h] >> 4) & 0x0F0F0F0Fu) << 3) + bias;   // chain 2k + 1 at byte k
        fv[h] = 0u;
        emin[h] = 0xFFFFFFFFu;
    }
    auto offset = [&](int h, int c) {
        return __builtin_amdgcn_ubfe((c & 1) ? oO[h] : oE[h], 8u * (uint32_t)(c >> 1), 8u) + (uint32_t)(c * kThc * 4);
    };
    auto chain = [&](int c) {
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const uint32_t e = A.half(h, c) - *(lds_u32*)(size_t)offset(h, c);
            fv[h] = __builtin_amdgcn_alignbit(fv[h], e, 31u);
            emin[h] = min(emin[h], e);
        }
    };
    // a unit with 8 slots has 5 to 8 chains: chains 0..4 are decided without
    // a test (in one block, so that their LDS reads are issued together)
#pragma unroll
    for (int c = kVbMaxChains - 1; c >= 5; --c)
        if (c < site.nch) chain(c);
#pragma unroll
    for (int c = 4; c >= 0; --c) chain(c);
#pragma unroll
    for (int h = 0; h < H; ++h) {
        fv[h] = act[h] ? fv[h] : 0u;
        fl[h] = *(lds_u32*)(size_t)(kSprOff + fv[h] * 4u);
    }
#pragma unroll
    for (int h = 0; h < H; ++h) {
        if (__builtin_amdgcn_ballot_w64(act[h] && emin[h] == 0u) != 0ull) {
            // A equals the high half of the threshold (those lanes did not flip
            // above): decide on the low half (rare: a loop, not unrolled)
            if (act[h] && emin[h] == 0u) {
#pragma unroll 1
                for (int c = 0; c < site.nch; ++c) {
                    const uint32_t off = offset(h, c);
                    const int32_t x = 15 - (int32_t)((off - (uint32_t)(c * kThc * 4)) >> 2);
                    if (site_half(site, kDomSweepHi, h, c) == *(lds_u32*)(size_t)off &&
                        site_half(site, kDomSweepLo, h, c) < gl(&site.up->thr_lo[c][0])[x])
                        fl[h] |= 1u << (4 * c);
                }
            }
        }
    }
}

// Where an adjacency entry points: with a complemented copy it is the word's LDS
// address above 5 bits of in-word shift, else a position and the sign of J.
template <int RPAD, bool CPL>
__device__ __forceinline__ void entry_word(uint32_t e, uint32_t sp_lds, uint32_t& ad, uint32_t& sh, uint32_t& sg)
{
    using S = Sl<RPAD>;
    if (CPL) {
        ad = e >> 5;
        sh = e;
        sg = 0u;
    } else {
        ad = sp_lds + S::boff(e);
        sh = e & (uint32_t)(S::P - 1);
        sg = (uint32_t)((int32_t)e >> 31);
    }
}

// The entry, or the own one in lanes past their degree (in 2.4-cycle operations
// and a bitop3: a comparison and a selection cost 8 to 25 cycles here).
__device__ __forceinline__ uint32_t entry_or_own(uint32_t e, uint32_t own, int32_t d, int32_t deg)
{
    const uint32_t m = (uint32_t)((int32_t)((uint32_t)d - (uint32_t)deg) >> 31);
    return (e & m) | (own & ~m);
}

template <int RPAD, bool CPL>
__device__ __forceinline__ uint32_t own_entry(int32_t q, const VbLds& L)
{
    using S = Sl<RPAD>;
    return CPL ? ((L.sp_lds + S::boff((uint32_t)q)) << 5) | ((uint32_t)q & (uint32_t)(S::P - 1)) : (uint32_t)q;
}

// Makes the entries past a lane's degree (up to the chunk's largest) the own one.
template <int RPAD, bool CPL, int NE, int H>
__device__ __forceinline__ void entries_ready(Stage<NE, H>& st, const VbChunk& T, int32_t q, const VbLds& L)
{
    // (a resident unit reads 4, 8 or 12 words whatever the degree)
    if (NE == kHbmMax && T.even()) return;
#pragma unroll
    for (int i = 0; i < NE / 4; ++i) {
        if (i == 0 || T.degree() > 4 * i) {
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const uint32_t own = own_entry<RPAD, CPL>(q + 64 * h, L);
#pragma unroll
                for (int j = 0; j < 4; ++j) st.e[h][i][j] = entry_or_own(st.e[h][i][j], own, 4 * i + j, st.deg[h]);
            }
        }
    }
}

// Counts of unsatisfied bonds of chunk T (positions q, q + 64) per chain: cA holds
// P-bit fields (for RPAD 8 while every degree of the chunk is below 16), else for
// RPAD 8 (true returned) cA / cB hold the even / odd chains in 8-bit fields.  The
// words of as many neighbours as the chunk's largest degree asks for, up to NE, are
// read together; the rest of longer rows follows four entries at a time.
// nbr(h, d, address, shift, sign): the word of entry d; own_ad, own_sh: the own one.
template <int RPAD, bool CPL, class PE, class WORD, int NE, int H>
__device__ __forceinline__ bool chunk_count(const Stage<NE, H>& E, const VbChunk& T, int32_t q, const VbLds& L, PE ent,
                                            WORD&& nbr, const uint32_t (&own_ad)[H], const uint32_t (&own_sh)[H],
                                            uint32_t (&cA)[H], uint32_t (&cB)[H])
{
    using S = Sl<RPAD>;
    typedef __attribute__((address_space(3))) uint32_t lds_u32;
    auto word = [&](uint32_t a) -> uint32_t { return *(const lds_u32*)(size_t)a; };
    uint32_t o0[H];
#pragma unroll
    for (int h = 0; h < H; ++h) cA[h] = cB[h] = 0u;
    auto sum = [&](auto nd) __attribute__((always_inline)) {
        constexpr int N = decltype(nd)::value;
        uint32_t w[H][N], sh[H][N], sg[H][N], ow[H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            ow[h] = word(own_ad[h]);
#pragma unroll
            for (int d = 0; d < N; ++d) {
                uint32_t ad;
                nbr(h, d, ad, sh[h][d], sg[h][d]);
                w[h][d] = word(ad);
            }
        }
#pragma unroll
        for (int h = 0; h < H; ++h) {
            o0[h] = ow[h] >> own_sh[h];
#pragma unroll
            for (int d = 0; d < N; ++d) cA[h] += ((w[h][d] >> (sh[h][d] & 31u)) ^ o0[h] ^ sg[h][d]) & S::M;
        }
        // (the cases stay apart: merged, their entries are read by a computed index
        // from private memory)
        asm volatile("" ::"n"(N));
    };
    const int32_t md = T.degree();
    if (NE > kHbmMax) {
        // (a resident unit's latency: few steps to the right case)
        if (md <= 4)
            sum(std::integral_constant<int, 4>{});
        else if (md <= 8)
            sum(std::integral_constant<int, 8>{});
        else
            sum(std::integral_constant<int, NE>{});
    } else {
        switch (md) {
            case 0:
            case 1: sum(std::integral_constant<int, 1>{}); break;
            case 2: sum(std::integral_constant<int, 2>{}); break;
            case 3: sum(std::integral_constant<int, 3>{}); break;
            case 4: sum(std::integral_constant<int, 4>{}); break;
            case 5: sum(std::integral_constant<int, 5>{}); break;
            case 6: sum(std::integral_constant<int, 6>{}); break;
            case 7: sum(std::integral_constant<int, 7>{}); break;
            default: sum(std::integral_constant<int, 8>{}); break;
        }
    }
    const bool wide = RPAD == 8 && md > 15;
    if (md > NE) {
        auto rest = [&](auto hc) __attribute__((always_inline)) {
            constexpr int h = decltype(hc)::value;
            const uint32_t own = own_entry<RPAD, CPL>(q + 64 * h, L), o = o0[h];
            const int32_t r0 = E.r0[h], deg = E.deg[h];
            uint32_t a = cA[h], b = 0u;
            if (wide) {
                b = (a >> 4) & 0x0F0F0F0Fu;
                a &= 0x0F0F0F0Fu;
            }
            for (int32_t d0 = NE; d0 < md; d0 += 4) {
                uint32_t en[4], w[4], sh[4], sg[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) en[i] = ent[(uint32_t)(d0 + i < deg ? r0 + d0 + i : r0)];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t ad;
                    entry_word<RPAD, CPL>(entry_or_own(en[i], own, d0 + i, deg), L.sp_lds, ad, sh[i], sg[i]);
                    w[i] = word(ad);
                }
                const uint32_t m = wide ? 0x01010101u : S::M;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t f = (w[i] >> (sh[i] & 31u)) ^ o ^ sg[i];
                    a += f & m;
                    if (RPAD == 8) b += wide ? (f >> 4) & 0x01010101u : 0u;
                }
            }
            cA[h] = a;
            cB[h] = b;
        };
        rest(std::integral_constant<int, 0>{});
        if constexpr (H > 1) rest(std::integral_constant<int, 1>{});
    }
    return wide;
}

// Decides the chunk and writes the flips back: every lane XORs its flips into its
// spin word.  Returns the lane's flips in spin-word form, the blocks' added up.
template <int RPAD, bool CPL, int H>
__device__ __forceinline__ uint32_t chunk_flip(const Site& site, const VbChunk& T, const VbLds& L, const Draws<RPAD, H>& A,
                                               const uint32_t (&cA)[H], const uint32_t (&cB)[H], bool wide,
                                               const int32_t (&deg)[H], const uint32_t (&own_ad)[H],
                                               const uint32_t (&own_sh)[H])
{
    typedef __attribute__((address_space(3))) uint32_t lds_u32;
    const int lane = (int)threadIdx.x & 63;
    bool act[H];
#pragma unroll
    for (int h = 0; h < H; ++h) act[h] = T.full() || in_class(T, 64 * h + lane);
    uint32_t fl[H];
    if constexpr (RPAD == 8) {
        if (!wide)
            vb_decide_compact<H>(site, A, cA, deg, act, fl);
        else
            vb_decide_full<RPAD, H>(site, L, A, cA, cB, deg, act, fl);
    } else {
        vb_decide_full<RPAD, H>(site, L, A, cA, cB, deg, act, fl);
    }
    uint32_t sum = 0u;
#pragma unroll
    for (int h = 0; h < H; ++h) {
        if (fl[h]) {
            const uint32_t f = fl[h] << own_sh[h];
            __atomic_fetch_xor((lds_u32*)(size_t)own_ad[h], f, __ATOMIC_RELAXED);
            if (CPL) __atomic_fetch_xor((lds_u32*)(size_t)(own_ad[h] + (L.cp_lds - L.sp_lds)), f, __ATOMIC_RELAXED);
        }
        sum += fl[h];
    }
    return sum;
}

// Split units: after a colour class, the members publish the words they
// changed (written through by the caller), meet at a device-scope barrier and read
// the class's words back, so that every member's LDS copy is complete before
// the next class.  The wait is bounded: a member that does not see all
// arrivals within kBarrierTicks of the 100 MHz real-time clock raises the
// unit's abort flag and the context's error bit, and every member stops.
constexpr uint64_t kBarrierTicks = 2000000000ull;

// What the exchanges of a split unit need of its descriptor, kept in scalar
// registers over the sweep loop: read at each use they come from memory again after
// every fence, four dependent reads in each of a sweep's 6 or 7 exchanges.  Measured,
// us per sweep, one graph of 65536 spins in 13 members: 6 chains 40.2 -> 35.3, 8 chains
// 43.8 -> 38.9, 2 chains 30.2 -> 28.6.  With one chain slot they are read at each use
// all the same: kept, the loop's code came out slower (pairs of 10^6 spins 443 -> 469,
// 13 members of 65536 28.7 and 28.7).
template <bool KEEP>
struct SplitRef {
    SG_G uint32_t* state_;
    uint32_t* bar_;
    int32_t words_, members_;
    __device__ __forceinline__ explicit SplitRef(const VbUnit* up)
    {
        if (KEEP) {
            state_ = gl(uniform(up->state));
            bar_ = uniform(up->bar);
            words_ = __builtin_amdgcn_readfirstlane(up->state_words);
            members_ = __builtin_amdgcn_readfirstlane(up->members);
        }
    }
    __device__ __forceinline__ SG_G uint32_t* state(const VbUnit* up) const { return KEEP ? state_ : gl(up->state); }
    __device__ __forceinline__ uint32_t* bar(const VbUnit* up) const { return KEEP ? bar_ : up->bar; }
    __device__ __forceinline__ int32_t words(const VbUnit* up) const { return KEEP ? words_ : up->state_words; }
    __device__ __forceinline__ int32_t members(const VbUnit* up) const { return KEEP ? members_ : up->members; }
};

template <int RPAD, bool KEEP>
__device__ bool vb_exchange(const VbUnit* __restrict__ up, const VbLds& L, const SplitRef<KEEP>& ref, int32_t lo,
                            int32_t hi, uint32_t target)
{
    using S = Sl<RPAD>;
    // One thread fences for the workgroup (as a grid barrier does): the
    // workgroup barrier orders every wavefront's write-through stores before
    // its device-scope release, and its device-scope acquire before the
    // read-back below.  (A fence in every wavefront wrote back and invalidated
    // the shared caches once per wavefront, slowing every workgroup on them.)
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t* bar = ref.bar(up);
        int32_t ab = 0;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __hip_atomic_fetch_add(bar, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t start = wall_clock64();
        while (__hip_atomic_load(bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            if (__hip_atomic_load(bar + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) {
                ab = 1;
                break;
            }
            if (wall_clock64() - start > kBarrierTicks) {
                __hip_atomic_store(bar + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                atomicOr(up->err, 4);
                ab = 1;
                break;
            }
            __builtin_amdgcn_s_sleep(1);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        L.flag[0] = ab;
    }
    __syncthreads();
    if (L.flag[0] != 0) return false;
    const SG_G uint32_t* gs = ref.state(up);
    const int32_t w0 = lo >> S::LP, w1 = hi > lo ? ((hi - 1) >> S::LP) : w0 - 1;
    // (eight loads of a thread in flight: one at a time, a class of 3 10^5 spins
    // waited ten times for HBM)
    const int32_t bd = (int32_t)blockDim.x;
    int32_t w = w0 + (int32_t)threadIdx.x;
    for (; w + 7 * bd <= w1; w += 8 * bd) {
        uint32_t v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = gs[w + j * bd];
#pragma unroll
        for (int j = 0; j < 8; ++j) L.sp[w + j * bd] = v[j];
    }
    uint32_t v[7];
#pragma unroll
    for (int j = 0; j < 7; ++j) v[j] = w + j * bd <= w1 ? gs[w + j * bd] : 0u;
#pragma unroll
    for (int j = 0; j < 7; ++j)
        if (w + j * bd <= w1) L.sp[w + j * bd] = v[j];
    __syncthreads();
    return true;
}

// A pass of Philox blocks: lane m draws group g of chain c for block i of a batch, m =
// (8 i + g) nch + c (lanes past the last block draw what nobody reads).
struct FillLane {
    uint32_t g, i, rep, inst;
};

__device__ __forceinline__ FillLane fill_lane(const VbLds& L, int lane, int32_t nch)
{
    const uint32_t mul = (65536u + (uint32_t)nch - 1u) / (uint32_t)nch;
    const uint32_t m = (uint32_t)lane;
    const uint32_t dq = (m * mul) >> 16;           // m / nch = 8 i + g
    const uint32_t c = m - dq * (uint32_t)nch;
    return FillLane{dq & 7u, min(dq >> 3, (uint32_t)(vb_batch_chunks(nch) - 1)), L.ri[2 * c], L.ri[2 * c + 1]};
}

__device__ __forceinline__ U4 fill_draw(const FillLane& fr, uint32_t base, uint32_t t, uint64_t key)
{
    return philox_stream(key, (base >> 3) + fr.g, t, kDomSweepHi, fr.rep, fr.inst);
}

__device__ __forceinline__ void fill_put(const VbLds& L, const U4& A, int wl, int lane)
{
    L.xch[wl * 64 + lane] = make_uint4(A.x, A.y, A.z, A.w);
    wave_sync();
}

template <int RPAD>
__device__ void vb_snapshot(const VbUnit* __restrict__ up, const uint32_t* __restrict__ sp, int k)
{
    using S = Sl<RPAD>;
    const int32_t wn = up->words_n, nch = up->nch, sw = up->state_words;
    for (int32_t idx = threadIdx.x; idx < nch * wn; idx += blockDim.x) {
        const int32_t c = idx / wn;
        const int32_t w = idx - c * wn;
        uint32_t bits = 0;
#pragma unroll
        for (int b = 0; b < 32 / S::P; ++b) {
            const int32_t wi = w * (32 / S::P) + b;
            const uint32_t v = wi < sw ? sp[wi] : 0u;
            const uint32_t f = S::P == 32 ? v : (v >> (c * S::P)) & ((1u << (S::P & 31)) - 1u);
            bits |= f << (b * S::P);
        }
        gl(up->snap[c])[(int64_t)k * wn + w] = bits;
    }
}

// cnt[c] += the set bits of d in chain c's field (chains c < nch)
template <int RPAD>
__device__ __forceinline__ void win_count(uint32_t* cnt, uint32_t d, int32_t nch)
{
    using S = Sl<RPAD>;
#pragma unroll
    for (int c = 0; c < RPAD; ++c)
        if (c < nch)
            cnt[c] += (uint32_t)__popc(d & (S::P == 32 ? 0xffffffffu : (((1u << (S::P & 31)) - 1u) << (c * S::P))));
}

typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// Adds the four words of d ^ e, bit by bit, to the bit-sliced counters
// (ones, twos) of a thread, and the carries of weight 4 to the per-chain
// counts cnt4 (carry-save adders: sum = a ^ b ^ c, carry = majority): one
// masked popcount per chain for four words instead of four.
__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c) { return (a & b) | (c & (a | b)); }

template <int RPAD>
__device__ __forceinline__ void win_add4(uint32_t& ones, uint32_t& twos, uint32_t* cnt4, v4u a, v4u b, int32_t nch)
{
    const v4u d = a ^ b;
    const uint32_t h1 = maj3(ones, d.x, d.y);
    ones ^= d.x ^ d.y;
    const uint32_t h2 = maj3(ones, d.z, d.w);
    ones ^= d.z ^ d.w;
    const uint32_t f = maj3(twos, h1, h2);
    twos ^= h1 ^ h2;
    win_count<RPAD>(cnt4, f, nch);
}

// cnt = 4 cnt4 + the counts of the planes (ones, twos), per chain
template <int RPAD>
__device__ __forceinline__ void win_fold(uint32_t* cnt, uint32_t ones, uint32_t twos, int32_t nch)
{
    uint32_t c1[RPAD], c2[RPAD];
#pragma unroll
    for (int c = 0; c < RPAD; ++c) {
        c1[c] = 0u;
        c2[c] = 0u;
    }
    win_count<RPAD>(c1, ones, nch);
    win_count<RPAD>(c2, twos, nch);
#pragma unroll
    for (int c = 0; c < RPAD; ++c) cnt[c] = 4u * cnt[c] + c1[c] + 2u * c2[c];
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v);

// Windowed correlation (the paper's estimator: C(t_w + t, t_w) averaged over
// minor-third intervals of t_w + t, ratio 2^(1/4); Results and discussion,
// and the SI section on the extrapolation to large sizes and times), at the
// end of the sweep that ends at time tau <= t_max: for every stored waiting
// time t_w < tau and every chain, the overlap sum_i s_i(tau) s_i(t_w) =
// n - 2 popcount(s(tau) xor s(t_w)) over the chain's fields, added to the
// chain's sum for the interval of tau.  The spin words at the waiting times
// are stored in the same sliced packing as the LDS words (rows of `ws4`
// 16-byte groups; the words past state_words are zero on both sides), so the
// XOR of two words holds every chain's disagreements; a thread adds them up
// bit-sliced (carry-save adders) and counts the chains' fields of the carry
// planes.  The work is cut into blocks of 64 groups of one waiting time's
// row, taken in (waiting time, block) order as contiguous ranges by the
// wavefronts of all members (lane l counts group 64 b + l of block b): a
// lane keeps adding into the same carry-save planes until its wavefront
// reaches the next waiting time, so the planes are folded and the wavefront
// sums formed once or twice per sweep instead of once per waiting time.  The
// stored words are streamed from HBM with 16-byte loads, four blocks in
// flight per lane.  At the waiting times each thread stores the groups
// i = tid + member * threads (mod members * threads); no thread reads another's
// stores.
template <int RPAD>
__device__ __attribute__((noinline)) void vb_window(const VbUnit* __restrict__ up, uint32_t sp_off,
                                                   uint32_t acc_off, int64_t tau, int32_t k_store)
{
    constexpr int U = 4;
    typedef __attribute__((address_space(3))) v4u lds_u4;
    typedef __attribute__((address_space(3))) uint32_t lds_u32;
    const lds_u4* sp4 = (const lds_u4*)(size_t)sp_off;
    lds_u32* wacc = (lds_u32*)(size_t)acc_off;
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63;
    const int32_t nch = up->nch;
    const int32_t sw4 = (up->state_words + 3) >> 2;
    // waiting times before tau: t_w = 0, and t_w = 2^(k-1) < tau for k >= 1
    const int32_t kv = min(up->kw, tau >= 2 ? 2 + (63 - __clzll((unsigned long long)(tau - 1))) : 1);
    const int32_t stride = nthr * up->members;
    const int32_t w0 = tid + up->member * nthr;
    SG_G v4u* ws4 = (SG_G v4u*)gl(up->wsnap);
    for (int i = tid; i < kv * RPAD; i += nthr) wacc[i] = 0u;
    __syncthreads();
    const int32_t nbr = (sw4 + 63) >> 6;   // blocks per row
    const int32_t nb = kv * nbr;
    const int32_t W = nthr >> 6;
    const int32_t gw = __builtin_amdgcn_readfirstlane(up->member * W + (tid >> 6));
    const int32_t GW = up->members * W;
    const int32_t per = (nb + GW - 1) / GW;
    const int32_t b0 = min(gw * per, nb), b1 = min(b0 + per, nb);
    const v4u zero = {0u, 0u, 0u, 0u};
    uint32_t cnt[RPAD];
#pragma unroll
    for (int c = 0; c < RPAD; ++c) cnt[c] = 0u;
    uint32_t ones = 0u, twos = 0u;   // bit-sliced counters
    int32_t kc = b0 / nbr;           // the waiting time being counted
    auto flush = [&](int32_t k) {
        win_fold<RPAD>(cnt, ones, twos, nch);
#pragma unroll
        for (int c = 0; c < RPAD; ++c) {
            if (c < nch) {
                const uint32_t v = wave_sum(cnt[c]);
                if (lane == 0 && v) atomicAdd((uint32_t*)&wacc[k * RPAD + c], v);
            }
            cnt[c] = 0u;
        }
        ones = twos = 0u;
    };
    for (int32_t b = b0; b < b1; b += U) {
        v4u a[U], w[U];
        int32_t kb[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t bb = b + u;
            const int32_t k = bb < b1 ? bb / nbr : kc;
            const int32_t g = (bb - k * nbr) * 64 + lane;
            const bool ok = bb < b1 && g < sw4;
            kb[u] = k;
            w[u] = ok ? ws4[(int64_t)k * sw4 + g] : zero;
            a[u] = ok ? sp4[g] : zero;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (b + u < b1) {
                if (kb[u] != kc) {
                    flush(kc);
                    kc = kb[u];
                }
                win_add4<RPAD>(ones, twos, cnt, a[u], w[u], nch);
            }
        }
    }
    if (b1 > b0) flush(kc);
    if (k_store >= 0) {
        SG_G v4u* dst = ws4 + (int64_t)k_store * sw4;
        for (int32_t i = w0; i < sw4; i += stride) dst[i] = sp4[i];
    }
    __syncthreads();
    const int32_t bin = vb_window_bin((uint64_t)tau);
    for (int i = tid; i < kv * nch; i += nthr) {
        const int32_t k = i / nch, c = i - k * nch;
        const long long o = (up->member == 0 ? (long long)up->n : 0ll) - 2ll * (long long)wacc[k * RPAD + c];
        atomicAdd((unsigned long long*)(up->win[c] + (int64_t)k * up->n_bins + bin), (unsigned long long)o);
    }
}

template <int RPAD, bool RES, bool SPLIT, bool CPL, int H, class PR, class PE, class PT>
__device__ void vb_loop(const VbUnit* __restrict__ up, const VbLds& L, PR row, PE ent, PT tab, const int32_t* cls,
                        int64_t t0, int32_t nsw, int64_t t_max, int lane, int wave, int W);

// (each variant is a function of its own so that its registers are
// allocated for it alone)
template <int RPAD, bool RES, bool SPLIT, bool CPL, int H>
__device__ __attribute__((noinline)) void vb_run(const VbUnit* __restrict__ up, uint32_t* smem_arr, uint32_t lds0,
                                                int64_t t0, int32_t nsw, int64_t t_max)
{
    // With fewer than 8 chain slots the dynamic LDS base is taken as a plain
    // offset: from the array itself this (called) function re-reads the base
    // from a per-kernel table at each use, and each re-read waits for all
    // outstanding LDS operations.  (With 8 slots the register the offset
    // would hold costs more than the re-reads: measured.)
    uint32_t* smem = RPAD == 8 ? smem_arr : (uint32_t*)(__attribute__((address_space(3))) uint32_t*)(size_t)lds0;
    const int tid = threadIdx.x, nthr = blockDim.x;
    // wave index made explicitly wave-uniform: the chunk cursor then lives in
    // scalar registers and class bounds come from scalar loads; a member of a
    // split unit numbers its wavefronts after those of the members before it
    const int Wl = nthr >> 6;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane((tid >> 6) + (SPLIT ? up->member * Wl : 0));
    const int W = SPLIT ? up->members * Wl : Wl;
    const int32_t sw = up->state_words, nch = up->nch, ncls = up->ncls;
    const VbLds L = vb_carve(smem, 0u, sw, nthr, nch, CPL);

    const SG_G uint32_t* gstate = gl(up->state);
    for (int32_t w = tid; w < sw; w += nthr) {
        const uint32_t v = gstate[w];
        L.sp[w] = v;
        if (CPL) L.cp[w] = ~v;
    }
    if (tid < ((sw + 3) & ~3) - sw) L.sp[sw + tid] = 0u;   // pad to 16 bytes (read by vb_window)
    // chain c's threshold high halves: word c kTab + j holds the entry for
    // x = 64 - j (0x10000 for x <= 0: always accepted)
    for (int i = tid; i < kVbMaxChains * kTab; i += nthr) {
        const int c = i / kTab, x = 64 - (i - c * kTab);
        L.thr[i] = x <= 0 ? 0x10000u : x < kVbXMax ? gl(&up->thr_hi[c][0])[x] : 0u;
    }
    // the same for |x| <= 15 in the compact tables: word c kThc + j holds the
    // entry for x = 15 - j
    for (int i = tid; i < kVbMaxChains * kThc; i += nthr) {
        const int c = i / kThc, x = 15 - (i - c * kThc);
        L.thc[i] = x <= 0 ? 0x10000u : gl(&up->thr_hi[c][0])[x];
    }
    for (int i = tid; i < 256; i += nthr) {
        uint32_t v = 0;
        for (int c = 0; c < 8; ++c) v |= (uint32_t)((i >> c) & 1) << (4 * c);
        L.spr[i] = v;
    }
    if (tid < kVbMaxChains) {
        L.accs[tid] = 0;
        L.ri[2 * tid] = up->rep[tid];
        L.ri[2 * tid + 1] = up->inst[tid];
    }
    for (int32_t k = tid; k <= ncls; k += nthr) L.cls[k] = gl(up->cls)[k];
    if (tid == 0) L.flag[0] = 0;   // chunks finished (split units: abort flag)
    const int32_t* cls = L.cls;
    __syncthreads();
    if constexpr (RES) {
        // row starts, and the entries in the form of vb_cpl_entries
        const int32_t n = up->n, m2 = up->m2;
        const SG_G int32_t* grow = gl(up->row);
        const SG_G uint32_t* gent = gl(up->ent);
        for (int32_t i = tid; i <= n; i += nthr) L.area[i] = grow[i];
        uint32_t* re = (uint32_t*)(L.area + n + 1);
        const uint32_t cofs = L.cp_lds - L.sp_lds;
        for (int32_t i = tid; i < m2 + kVbEntPad; i += nthr) {
            const uint32_t en = i < m2 ? gent[i] : 0u;
            re[i] = ((L.sp_lds + Sl<RPAD>::boff(en) + ((int32_t)en < 0 ? cofs : 0u)) << 5) | (en & (uint32_t)(Sl<RPAD>::P - 1));
        }
        // the chunks of the sweep, after the entries
        int32_t* tab = (int32_t*)(re + m2 + kVbEntPad);
        const SG_G int32_t* gtab = (const SG_G int32_t*)gl(up->chunk);
        for (int32_t i = tid; i < 4 * up->chunks; i += nthr) tab[i] = gtab[i];
        __syncthreads();
        vb_loop<RPAD, true, false, CPL, H>(up, L, (const int32_t*)L.area, (const uint32_t*)re, (const VbChunk*)tab, cls, t0, nsw,
                                        t_max, lane, wave, W);
    } else {
        // (wave-uniform addresses: the rows and entries are addressed by a scalar
        // base and 32-bit offsets, and the chunk records, in constant memory, come
        // by scalar loads, which do not wait for the entries in flight)
        vb_loop<RPAD, false, SPLIT, CPL, H>(up, L, gl(uniform(up->row)), gl(uniform(CPL ? up->entc : up->ent)),
                                         (const __attribute__((address_space(4))) VbChunk*)uniform(up->chunk), cls, t0, nsw,
                                         t_max, lane, wave, W);
    }
    // (split units keep `state` current by writing through)
    if (!SPLIT)
        for (int32_t w = tid; w < sw; w += nthr) gl(up->state)[w] = L.sp[w];
    __syncthreads();
    if (tid < nch) atomicAdd(up->accepted[tid], L.accs[tid]);
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += (uint32_t)__shfl_xor((int)v, o);
    return v;
}

// Accepted flips of one wavefront, counted per lane in the flips' own
// spin-word fields (n += flips of each chunk, of H blocks).  A P-bit field holds the
// flips of at most 2^P - 1 blocks: with 8 chain slots (4-bit fields) the counts move
// to byte fields (e: even chains, o: odd chains, chain c at byte c / 2) before a
// chunk could pass 15 blocks, and 17 such moves fill a byte; byte and 16-bit fields
// are summed over the wavefront into the unit's LDS totals before a chunk could pass
// 255 (65535) blocks, and every field at the end of each stretch of sweeps.
template <int RPAD>
struct VbAcc {
    uint32_t n = 0, e = 0, o = 0;   // per lane
    int32_t cn = 0, cb = 0;         // wave-uniform: blocks since the last fold (flush), folds since the last flush
};

template <int RPAD>
__device__ __forceinline__ void acc_fold(VbAcc<RPAD>& a)
{
    if (RPAD == 8) {
        a.e += a.n & 0x0F0F0F0Fu;
        a.o += (a.n >> 4) & 0x0F0F0F0Fu;
        a.n = 0u;
    }
    a.cn = 0;
}

template <int RPAD>
__device__ __forceinline__ void acc_flush(VbAcc<RPAD>& a, const VbLds& L, int32_t nch)
{
    const int lane = threadIdx.x & 63;
    // chain sums in 16-bit halves (at most 64 x 255 each) or whole words
    auto put = [&](int c, uint32_t v) {
        if (lane == 0 && c < nch && v != 0u) atomicAdd(&L.accs[c], (unsigned long long)v);
    };
    if (RPAD == 8) {
        const uint32_t e0 = wave_sum(a.e & 0x00FF00FFu), e1 = wave_sum((a.e >> 8) & 0x00FF00FFu);
        const uint32_t o0 = wave_sum(a.o & 0x00FF00FFu), o1 = wave_sum((a.o >> 8) & 0x00FF00FFu);
        put(0, e0 & 0xFFFFu);
        put(4, e0 >> 16);
        put(2, e1 & 0xFFFFu);
        put(6, e1 >> 16);
        put(1, o0 & 0xFFFFu);
        put(5, o0 >> 16);
        put(3, o1 & 0xFFFFu);
        put(7, o1 >> 16);
        a.e = 0u;
        a.o = 0u;
    } else if (RPAD == 4) {
        const uint32_t s0 = wave_sum(a.n & 0x00FF00FFu), s1 = wave_sum((a.n >> 8) & 0x00FF00FFu);
        put(0, s0 & 0xFFFFu);
        put(2, s0 >> 16);
        put(1, s1 & 0xFFFFu);
        put(3, s1 >> 16);
        a.n = 0u;
    } else if (RPAD == 2) {
        put(0, wave_sum(a.n & 0xFFFFu));
        put(1, wave_sum(a.n >> 16));
        a.n = 0u;
    } else {
        put(0, wave_sum(a.n));
        a.n = 0u;
    }
    a.cn = 0;
    a.cb = 0;
}

// (fl: the flips of H blocks added up)
template <int RPAD, int H>
__device__ __forceinline__ void acc_add(VbAcc<RPAD>& a, uint32_t fl, const VbLds& L, int32_t nch)
{
    a.n += fl;
    a.cn += H;
    if (RPAD == 8) {
        if (a.cn > 15 - H) {
            acc_fold(a);
            if (++a.cb == 17) acc_flush(a, L, nch);
        }
    } else if (RPAD == 4) {
        if (a.cn > 255 - H) acc_flush(a, L, nch);
    } else if (RPAD == 2) {
        if (a.cn > 65535 - H) acc_flush(a, L, nch);
    }
}

// The end of a sweep: snapshot at a grid time, windowed correlation.
template <int RPAD, bool SPLIT>
__device__ __forceinline__ void vb_sweep_end(const VbUnit* __restrict__ up, const VbLds& L, int64_t tn, int64_t t_max)
{
    const bool grid = tn <= t_max && (tn & (tn - 1)) == 0;
    const int32_t kn = grid ? 1 + (63 - __clzll((unsigned long long)tn)) : -1;
    if (grid) {
        if (!SPLIT || up->member == 0) vb_snapshot<RPAD>(up, L.sp, kn);
        __syncthreads();
    }
    if (up->kw > 0 && tn <= t_max) {
        vb_window<RPAD>(up, L.sp_lds, L.sp_lds + (uint32_t)((const char*)L.wacc - (const char*)L.sp), tn,
                        kn < up->kw ? kn : -1);
        __syncthreads();
    }
}

// The sweep loop of one unit, or of one member of a split unit (`wave` and `W` then
// count the wavefronts of all members), for an adjacency in HBM or (RES) in LDS.
//
// The chunks of a sweep are numbered through its colour classes and dealt to the
// wavefronts in turn.  A chunk waits until every chunk of the classes before it is
// finished: the wavefronts meet at no barrier but at a counter of finished chunks
// in LDS, and take their chunks in order, so the lowest unfinished one never waits
// for another and every wait ends.  (Members of a split unit meet at a barrier
// after every class, where they exchange spin words.)
//
// Everything that does not depend on spins is done before the wait: the entries of
// the chunk after it and the rows of the one after that are requested, the chunk's
// random numbers drawn and its neighbours' addresses formed.  After the wait all
// spin words are read at once, counted and decided, and the flips written back.
// That matters in both regimes: a single wavefront issues an instruction about
// every 8 cycles whatever else runs, so a small unit is bound by the instructions
// between the last flip of a class and the first read of the next, and with 4
// wavefronts a SIMD a large one is bound by exposed latency as much as by issue.  So
// a large unit's chunk has H = 2 blocks, whose latencies overlap (a resident one's has
// one: fewer instructions between two classes; split_chunk_blocks for split ones), and chunks of one degree (most:
// positions are sorted by it inside a class) need no rows, no masks and exactly as
// many reads as neighbours.
//
// Measured, us per sweep, against one barrier per class, one block per chunk and one
// masked LDS round trip per neighbour: 256 graphs of 65536 spins with 6 chains 72.9
// (90.0: 139 VALU, 108 SALU and 25 LDS instructions a block, 4 wavefronts a SIMD; with
// one block a chunk 85.7), 1 chain 48.6 (70.1; 5.5 TB/s of adjacency), 2 chains 54.1
// (72.8), 4 chains 68.0 (83.2); one unit of 10^6 spins and 1 chain 560 (813).  One
// resident unit of 1024 spins and 2 chains 2.2 (8.3; the time from counter to
// counter, about 1000 cycles for each of 5 classes; 2.06 in a loop of its own, which
// went when the streamed units' loop became this one), 2048 of them 12 (27).
template <int RPAD, bool RES, bool SPLIT, bool CPL, int H, class PR, class PE, class PT>
__device__ void vb_loop(const VbUnit* __restrict__ up, const VbLds& L, PR row, PE ent, PT tab, const int32_t* cls,
                        int64_t t0, int32_t nsw, int64_t t_max, int lane, int wave, int W)
{
    typedef __attribute__((address_space(3))) uint32_t lds_u32;
    const int tid = threadIdx.x;
    up = uniform(up);
    // The unit's scalars arrive through a pointer argument, which the
    // compiler cannot take as uniform: made explicitly wave-uniform, the
    // per-chain tests and the sweep loop branch on scalar registers instead
    // of masking lanes
    const int32_t nchains = __builtin_amdgcn_readfirstlane(up->nch), ncls = __builtin_amdgcn_readfirstlane(up->ncls);
    const int32_t chunks = __builtin_amdgcn_readfirstlane(up->chunks);
    nsw = __builtin_amdgcn_readfirstlane(nsw);
    W = __builtin_amdgcn_readfirstlane(W);
    t0 = uniform64(t0);
    t_max = uniform64(t_max);
    // the Philox key is the same for every lane: kept in scalar registers,
    // so that the per-round keys cost no vector registers
    const uint64_t unit_key = (uint64_t)uniform64((int64_t)up->key);
    const bool win = __builtin_amdgcn_readfirstlane(up->kw) > 0;
    const int wl = __builtin_amdgcn_readfirstlane(tid >> 6);   // wavefront inside the workgroup
    lds_u32* const fin = (lds_u32*)(uint32_t*)L.flag;
    constexpr int NE = RES ? kLdsMax : kHbmMax;
    static_assert(H == 2 || (H == 1 && (RES || (SPLIT && RPAD == 8))), "the variants there are");
    // (wavefronts past the chunks of a sweep only take part in its end)
    const int32_t step = min(W, chunks);
    const int32_t B = vb_batch_chunks(nchains);

    auto tab_at = [&](int32_t id) -> VbChunk {
        VbChunk T;
        T.a = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)tab[id].a);
        T.b = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)tab[id].b);
        T.r0 = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)tab[id].r0);
        return T;
    };
    auto wrap = [&](int32_t& id) {
        const bool over = id >= chunks;
        id -= over ? chunks : 0;
        return over;
    };
    VbAcc<RPAD> acc;
    // this wavefront's current chunk and its sweep; the sweep the unit is in, its
    // first chunk's number and (split units) the class the members are in
    int32_t id = min(wave, chunks - 1), cs = wave < step ? 0 : nsw;
    int32_t s = 0, k = 0;
    uint32_t first = 0u;
    // split units: this wavefront's chunks of the class, the first one's base; their
    // words are written through to HBM together at the end of the class (a store per
    // chunk would be waited for with the next chunk's entries)
    int32_t own_n = 0, own_base = 0;
    const SplitRef<SPLIT && (RPAD > 1)> ref(up);
    auto exchange = [&]() {
        using S = Sl<RPAD>;
        constexpr int LW = 6 + (H - 1) - S::LP;   // log2 of a chunk's words
        for (int32_t i = lane; i < own_n << LW; i += 64) {
            const uint32_t wi = ((uint32_t)(own_base + (i >> LW) * step * 64 * H) >> S::LP) + (uint32_t)(i & ((1 << LW) - 1));
            if (wi < (uint32_t)ref.words(up)) ref.state(up)[wi] = L.sp[wi];
        }
        own_n = 0;
        const int32_t lo = cls_at(cls, k), hi = cls_at(cls, k + 1);
        ++k;
        return vb_exchange<RPAD>(up, L, ref, lo, hi, (uint32_t)ref.members(up) * (uint32_t)(s * ncls + k));
    };
    // ends the sweeps before `to`
    auto sweeps = [&](int32_t to) -> bool {
        while (s < to) {
            if (SPLIT) {
                while (k < ncls)
                    if (!exchange()) return false;
                k = 0;
            }
            ++s;
            first += (uint32_t)chunks;
        }
        return true;
    };

    // The sweeps are run in stretches up to one after which all wavefronts meet for a
    // snapshot or the windowed sums.  Nothing but scalars lives from one stretch to
    // the next (the lane number is opaque in each, so that what follows from it is
    // not kept either): no vector register is held, or spilled, over those calls.
    for (;;) {
        int32_t stop = nsw;
        {
            const int64_t tn = t0 + s + 1;
            const int64_t te = win || tn <= 1 ? tn : (int64_t)1 << (64 - __clzll((unsigned long long)(tn - 1)));
            if (te <= t_max && te - t0 < nsw) stop = (int32_t)(te - t0);
        }
        if (cs < stop) {
            int ln = lane;
            asm volatile("" : "+v"(ln));
            const FillLane fr = fill_lane(L, ln, nchains);
            const uint32_t* xg = (const uint32_t*)(L.xch + wl * 64) + (uint32_t)(ln >> 3) * (uint32_t)nchains * 4u + (((uint32_t)ln & 7u) >> 1);
            // the next chunk and the one after (a chunk's record is read two chunks ahead)
            int32_t id2 = id;
            VbChunk T0 = tab_at(id), T1, T2;
            id2 += step;
            wrap(id2);
            T1 = tab_at(id2);
            id2 += step;
            wrap(id2);
            T2 = tab_at(id2);
            // batches of several chunks (fewer than 5 chains): position and sweep of this
            // lane's block of the next batch
            int32_t bi = B, f_id = 0, f_base = 0;
            uint32_t f_t = 0u;
            auto ahead = [&](int32_t fid, uint32_t t) {
                f_id = fid;
                f_t = t;
                while (f_id >= chunks) {
                    f_id -= chunks;
                    ++f_t;
                }
                f_base = VbChunk{tab[f_id].a, 0u, 0u, 0u}.base() + 64 * (H > 1 ? (int32_t)fr.i & 1 : 0);
            };
            // E holds the rows and entries of the current chunk (in flight), R the rows of
            // the next one
            Stage<NE, H> E, R;
            auto request = [&]() __attribute__((always_inline)) {
                // (past the last chunk of the launch these re-read entries that are not
                // used: no branch)
                rows_ready(E, R, T0, ln);
                load_ents(ent, E, T0.degree());
                load_rows(row, T1, ln, R);
            };
            auto one = [&]() __attribute__((always_inline)) -> bool {
                const VbChunk T = T0;
                // (opaque: the tests of chain numbers stay scalar comparisons here and the
                // round keys are formed here, instead of being kept, and spilled, across the
                // loop)
                int32_t nch = nchains;
                uint64_t key = unit_key;
                asm volatile("" : "+s"(nch), "+s"(key));
                const uint32_t t = (uint32_t)t0 + (uint32_t)s;
                const int32_t q = T.base() + ln;
                T0 = T1;
                T1 = T2;
                id2 += step;
                wrap(id2);
                T2 = tab_at(id2);
                Draws<RPAD, H> A;
                {
                    auto take = [&](int h, int block) __attribute__((always_inline)) {
                        const uint32_t* gx = xg + (uint32_t)block * 32u * (uint32_t)nch;
#pragma unroll
                        for (int c = 0; c < RPAD; ++c)
                            if (c <= RPAD / 2 || c < nch) A.a[h][c] = ((const uint16_t*)(gx + 4 * c))[ln & 1];
                    };
                    if (RPAD == 8) {
                        // one block a pass: both passes are drawn together, then go through
                        // the same LDS in turn, the first block's last
                        U4 d[H];
#pragma unroll
                        for (int h = 0; h < H; ++h) d[h] = fill_draw(fr, (uint32_t)T.base() + 64u * (uint32_t)h, t, key);
                        fill_put(L, d[H - 1], wl, ln);
                        take(0, 0);
                        if (H == 2) {
                            wave_sync();
                            fill_put(L, d[0], wl, ln);
                            A.first = (const uint16_t*)xg + (ln & 1);
                        }
                    } else {
                        if (bi >= B) {
                            fill_put(L, fill_draw(fr, (uint32_t)f_base, f_t, key), wl, ln);
                            bi = 0;
                            ahead(f_id + B / H * step, f_t);
                        }
#pragma unroll
                        for (int h = 0; h < H; ++h) take(h, bi + h);
                        bi += H;
                    }
                }
                uint32_t own_ad[H], own_sh[H];
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    own_ad[h] = L.sp_lds + Sl<RPAD>::boff((uint32_t)(q + 64 * h));
                    own_sh[h] = (uint32_t)(q + 64 * h) & (uint32_t)(Sl<RPAD>::P - 1);
                }
                entries_ready<RPAD, CPL>(E, T, q, L);
                // (a resident unit's latency is the time from the wait on: addresses before it)
                uint32_t ad[RES ? NE : 1];
                if (RES) {
#pragma unroll
                    for (int d = 0; d < NE; ++d) {
                        ad[RES ? d : 0] = E.e[0][d >> 2][d & 3] >> 5;
                        asm volatile("" : "+v"(ad[RES ? d : 0]));   // (not after the wait)
                    }
                }
                if (SPLIT) {
                    while (k < T.cls())
                        if (!exchange()) return false;
                } else {
                    const uint32_t need = first + (uint32_t)T.before();
                    uint32_t done;
                    while ((int32_t)((done = __builtin_amdgcn_readfirstlane(*(volatile lds_u32*)fin)) - need) < 0) {}
                    wave_sync();
                    if (RES) {
                        __builtin_amdgcn_s_setprio(3);
                    } else {
                        // The scheduler prefers the oldest of a SIMD's wavefronts,
                        // which would run ahead and wait at the end of each class (1640
                        // cycles a chunk, the youngest 300): the wavefronts behind
                        // the unit's average get the higher priority
                        const int32_t behind = (int32_t)(done - first) - id;
                        if (behind > 0)
                            __builtin_amdgcn_s_setprio(3);
                        else if (behind > -4)
                            __builtin_amdgcn_s_setprio(2);
                        else if (behind > -8)
                            __builtin_amdgcn_s_setprio(1);
                        else
                            __builtin_amdgcn_s_setprio(0);
                    }
                }
                uint32_t cA[H], cB[H];
                auto nbr = [&](int h, int d, uint32_t& a, uint32_t& sh, uint32_t& sg) __attribute__((always_inline)) {
                    entry_word<RPAD, CPL>(E.e[h][d >> 2][d & 3], L.sp_lds, a, sh, sg);
                    if (RES) a = ad[RES ? d : 0];
                };
                const bool wide = chunk_count<RPAD, CPL>(E, T, q, L, ent, nbr, own_ad, own_sh, cA, cB);
                int32_t deg[H];
#pragma unroll
                for (int h = 0; h < H; ++h) deg[h] = E.deg[h];
                // the entries have been used: the next chunk's are requested here (HBM), or
                // once the chunk is finished (LDS: a resident unit's wait is over sooner)
                if (!RES) request();
                const uint32_t fl = chunk_flip<RPAD, CPL, H>(Site{up, key, t, q, nch}, T, L, A, cA, cB, wide, deg, own_ad, own_sh);
                wave_sync();
                if (SPLIT) {
                    own_base = own_n == 0 ? T.base() : own_base;
                    ++own_n;
                } else {
                    // (the LDS operations of a wavefront take effect in order)
                    if (ln == 0) __atomic_fetch_add(fin, 1u, __ATOMIC_RELAXED);
                    if (RES) __builtin_amdgcn_s_setprio(0);
                    wave_sync();
                }
                if (RES) request();
                acc_add<RPAD, H>(acc, fl, L, nch);
                id += step;
                if (wrap(id) && ++cs < stop) return sweeps(cs);
                return true;
            };
            if (RPAD < 8) ahead(id + (int32_t)fr.i / H * step, (uint32_t)t0 + (uint32_t)cs);
            load_rows(row, T0, ln, R);
            rows_ready(E, R, T0, ln);
            load_ents(ent, E, T0.degree());
            load_rows(row, T1, ln, R);
            do {
                if (!one()) return;
            } while (cs < stop);
        }
        if (!sweeps(stop)) return;
        acc_fold(acc);
        acc_flush(acc, L, nchains);
        const int64_t tn = t0 + stop;
        if (tn <= t_max && (win || (tn & (tn - 1)) == 0)) {
            if (!SPLIT) __syncthreads();
            vb_sweep_end<RPAD, SPLIT>(up, L, tn, t_max);
        }
        if (stop >= nsw) break;
    }
    __syncthreads();
}

// t0p: device-resident number of sweeps done before this launch (read once;
// the counter is advanced by vb_advance_kernel after every launch group), so
// a captured graph of the sweep loop can be replayed unchanged.
__global__ void __launch_bounds__(1024) vb_sweep_kernel(const VbUnit* __restrict__ units,
                                                        const int64_t* __restrict__ t0p,
                                                        int32_t nsw, int64_t t_max)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t smem[];
    uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) uint32_t*)smem;
    const VbUnit* up = (const VbUnit*)(gl(units) + blockIdx.x);
    // The sweep functions read the spin words at LDS offset 0, where the
    // dynamic array starts in a kernel that declares no static LDS (a
    // constant test: a build where that does not hold reports an error)
    if (lds0 != 0u) {
        if (threadIdx.x == 0) atomicOr(up->err, 8);
        return;
    }
    asm volatile("" : "+s"(lds0));   // an opaque value: the callee cannot re-derive it from the array
    const int64_t t0 = *gl(t0p);
    if (up->resident) {
        switch (up->rpad) {
            case 1: vb_run<1, true, false, true, 1>(up, smem, lds0, t0, nsw, t_max); break;
            case 2: vb_run<2, true, false, true, 1>(up, smem, lds0, t0, nsw, t_max); break;
            case 4: vb_run<4, true, false, true, 1>(up, smem, lds0, t0, nsw, t_max); break;
            default: vb_run<8, true, false, true, 1>(up, smem, lds0, t0, nsw, t_max); break;
        }
    } else if (up->members > 1) {
        switch (up->rpad) {
            case 1: vb_run<1, false, true, false, 2>(up, smem, lds0, t0, nsw, t_max); break;
            case 2: vb_run<2, false, true, false, 2>(up, smem, lds0, t0, nsw, t_max); break;
            case 4: vb_run<4, false, true, false, 2>(up, smem, lds0, t0, nsw, t_max); break;
            default:
                if (up->blocks == 1)
                    vb_run<8, false, true, false, 1>(up, smem, lds0, t0, nsw, t_max);
                else
                    vb_run<8, false, true, false, 2>(up, smem, lds0, t0, nsw, t_max);
                break;
        }
    } else if (up->cpl) {
        switch (up->rpad) {
            case 1: vb_run<1, false, false, true, 2>(up, smem, lds0, t0, nsw, t_max); break;
            case 2: vb_run<2, false, false, true, 2>(up, smem, lds0, t0, nsw, t_max); break;
            case 4: vb_run<4, false, false, true, 2>(up, smem, lds0, t0, nsw, t_max); break;
            default: vb_run<8, false, false, true, 2>(up, smem, lds0, t0, nsw, t_max); break;
        }
    } else {
        switch (up->rpad) {
            case 1: vb_run<1, false, false, false, 2>(up, smem, lds0, t0, nsw, t_max); break;
            case 2: vb_run<2, false, false, false, 2>(up, smem, lds0, t0, nsw, t_max); break;
            case 4: vb_run<4, false, false, false, 2>(up, smem, lds0, t0, nsw, t_max); break;
            default: vb_run<8, false, false, false, 2>(up, smem, lds0, t0, nsw, t_max); break;
        }
    }
}

__global__ void vb_advance_kernel(int64_t* t, int32_t nsw, uint32_t* bars, int n_bar)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *t += nsw;
    for (int i = threadIdx.x; i < n_bar; i += blockDim.x) bars[i] = 0u;
}

// Initial configurations and the t = 0 snapshot.
__global__ void __launch_bounds__(1024) vb_init_kernel(const VbUnit* __restrict__ units)
{
    const VbUnit* up = units + blockIdx.x;
    if (up->member != 0) return;   // members of a split unit share its state
    const int32_t n = up->n, wn = up->words_n, nch = up->nch, rpad = up->rpad;
    for (int32_t idx = threadIdx.x; idx < nch * wn; idx += blockDim.x) {
        const int32_t c = idx / wn;
        const int32_t w = idx - c * wn;
        uint32_t bits;
        if (up->init_mode[c] == 0) {
            const U4 o = philox_stream(up->seed[c], (uint32_t)(w >> 2), 0u, kDomInit, up->rep[c],
                                       up->inst[c]);
            bits = word_of(o, (uint32_t)(w & 3));
        } else if (up->init_mode[c] == 1) {
            bits = 0;
        } else {
            bits = up->given[c][w];
        }
        const int32_t pe = n - 32 * w;
        if (pe < 32) bits &= (1u << pe) - 1u;
        up->snap[c][w] = bits;
    }
    __syncthreads();
    const VbLayout lay(rpad);
    for (int32_t w = threadIdx.x; w < up->state_words; w += blockDim.x) {
        const int32_t p0 = w * lay.P;   // first position of the word
        uint32_t word = 0;
        for (int32_t c = 0; c < nch; ++c) {
            const uint32_t v = up->snap[c][p0 >> 5];
            const uint32_t f = lay.P == 32 ? v : (v >> (p0 & 31)) & ((1u << lay.P) - 1u);
            word |= f << (c * lay.P);
        }
        up->state[w] = word;
        if (up->kw > 0) up->wsnap[w] = word;   // the waiting time t_w = 0
    }
}

}  // namespace

size_t vb_resident_bytes(int32_t n, int32_t m2, int32_t ncls)
{
    // row starts, entries, chunks (a class boundary inside a block of 64 positions adds one)
    const size_t chunks = (size_t)n / 64 + 1 + (size_t)ncls;
    return ((size_t)(n + 1 + m2 + kVbEntPad) * 4 + chunks * sizeof(VbChunk) + 15) & ~(size_t)15;
}

size_t vb_lds_bytes(int32_t n, int32_t rpad, int32_t nch, int threads, bool cpl)
{
    const size_t sw = (size_t)VbLayout(rpad).words(n);
    const size_t waves = (size_t)threads / 64;
    return kSpOff + ((sw + 3) & ~(size_t)3) * 4 * (cpl ? 2 : 1) + (size_t)kVbMaxChains * kTab * 4 + kVbMaxChains * 8 + 16 +
           (kMaxCls + 4) * 4 + kVbMaxChains * 8 + (size_t)kMaxGrid * kVbMaxChains * 4 + waves * 64 * 16;
}

void vb_cpl_entries(const uint32_t* ent, size_t m, size_t pad, int32_t rpad, int32_t n, uint32_t* out)
{
    const VbLayout lay(rpad);
    const uint32_t swp = ((uint32_t)lay.words(n) + 3u) & ~3u;
    for (size_t e = 0; e < m + pad; ++e) {
        const uint32_t en = e < m ? ent[e] : 0u;
        const uint32_t pos = en & 0x7fffffffu;
        const uint32_t addr = kSpOff + 4u * (pos / (uint32_t)lay.P) + ((en >> 31) != 0u ? 4u * swp : 0u);
        out[e] = (addr << 5) | (pos % (uint32_t)lay.P);
    }
}

hipError_t vb_init(const VbUnit* units, int n_units, int threads, size_t, hipStream_t s)
{
    if (n_units <= 0) return hipSuccess;
    hipLaunchKernelGGL(vb_init_kernel, dim3(n_units), dim3(threads), 0, s, units);
    return hipGetLastError();
}

hipError_t vb_prepare()
{
    // set once (thread-safe initialisation of a local static)
    static const hipError_t attr = hipFuncSetAttribute((const void*)vb_sweep_kernel,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return attr;
    return hipSuccess;
}

hipError_t vb_sweep(const VbUnit* units, int n_units, int threads, size_t lds_bytes, const int64_t* t0p,
                    int32_t n_sweeps, int64_t t_max, hipStream_t s)
{
    if (n_units <= 0 || n_sweeps <= 0) return hipSuccess;
    hipLaunchKernelGGL(vb_sweep_kernel, dim3(n_units), dim3(threads), lds_bytes, s, units, t0p,
                       n_sweeps, t_max);
    return hipGetLastError();
}

hipError_t vb_advance(int64_t* t, int32_t n_sweeps, uint32_t* bars, int n_bar, hipStream_t s)
{
    hipLaunchKernelGGL(vb_advance_kernel, dim3(1), dim3(256), 0, s, t, n_sweeps, bars, n_bar);
    return hipGetLastError();
}

}  // namespace sg
