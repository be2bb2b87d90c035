// Internal device-side descriptors and kernel launchers shared by the host
// runtime (sg_host.cpp) and the HIP kernels (sg_vb.hip, sg_vbm.hip,
// sg_sk.hip, sg_skg.hip, sg_measure.hip).  Not part of the public interface.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sg_stage.h"
#include "sg_vb_unit.h"

namespace sg {

constexpr int kWindowBinsMax = 128;  // minor-third intervals of times below 2^32
constexpr size_t kMeasureScratchElems = (size_t)1 << 20;   // int64 staging of sg_measure_noalloc (8 MiB)

// A multispin VB work unit (sg_vbm.hip): one graph and up to 64 chains on it,
// each with its own couplings, temperature and random numbers, packed as the
// bits of one 64-bit word per vertex (the paper's multispin coding: Methods;
// SI bipartite-graph section).  The spins stay in LDS during a launch.
constexpr int kVbmChains = 64;
constexpr int kVbmMaxN = 16384;    // n 64-bit words must fit in LDS
struct VbmUnit {
    const int32_t* row;        // [n+1] adjacency row starts, sweep order
    const uint32_t* ent;       // [2m + kVbEntPad] neighbour position in bits 0..30 (bit 31 ignored)
    const uint64_t* jw;        // [2m + kVbEntPad] bit c: chain c's coupling on the entry is -1
    const int32_t* cls;        // [ncls+1] first position of each colour class
    uint64_t* state;           // [n] spin words between launches (bit c: chain c's spin is -1)
    const uint32_t* thr;       // [2][64][kVbXMax]: chain c's thr[x] >> 16 (0..65536), then thr[x] & 0xffff
                               // (entry x = 0 unused)
    uint64_t key;              // Philox key (seed) shared by every chain of the unit
    uint32_t* snap[kVbmChains];
    unsigned long long* accepted[kVbmChains];
    uint32_t inst[kVbmChains];
    uint32_t rep[kVbmChains];
    int32_t n;
    int32_t ncls;
    int32_t nch;
    int32_t words_n;           // ceil(n / 32)
    int32_t init_mode[kVbmChains];
    const uint32_t* given[kVbmChains];
    uint64_t seed;
};

// SK couplings as bits, by block columns of 64 spins: bit j of word k of block b
// is 1 where the coupling of spins k and 64 b + j is -1 (0 on the diagonal and
// past n).  The number of blocks is even, and a spin's words of blocks 2 p and 2 p
// + 1 are neighbours (one 16-byte load).
__host__ __device__ __forceinline__ int32_t sk_blocks(int32_t n) { return 2 * ((n + 127) >> 7); }
__host__ __device__ __forceinline__ int64_t sk_word(int32_t n_blocks, int64_t b, int64_t k)
{
    return ((b >> 1) * 64 * n_blocks + k) * 2 + (b & 1);
}

// Real couplings: floats from one row to the next on the device.
__host__ __device__ __forceinline__ int32_t skg_pitch(int32_t n) { return (n + 255) & ~255; }

// The chain that workgroup `bid` of a launch of one workgroup per chain runs:
// workgroups go to the 8 XCDs in turn, and the chains of an XCD are consecutive,
// so that the replicas of a sample, which read the same couplings, share an L2.
__device__ __forceinline__ int32_t chain_of_block(int32_t bid, int32_t n_chains)
{
    const int32_t x = bid & 7, i = bid >> 3, q = n_chains >> 3, r = n_chains & 7;
    return x * q + min(x, r) + i;
}

// One SK chain (a replica of an instance).
struct SkChain {
    const uint64_t* Jw;        // coupling words, see sk_word
    uint32_t* state;           // [words_n] position-order bits (1 = spin -1)
    int32_t* H;                // [n] local fields between launches
    uint32_t* snap;            // [K][words_n]
    unsigned long long* accepted;
    const uint64_t* thr;       // [thr_len] thresholds (uint64), x < thr_len
    uint64_t seed;
    uint32_t inst;
    uint32_t rep;
    int32_t n;
    int32_t words_n;
    int32_t thr_len;           // thr[x] == 0 for x >= thr_len
    int32_t init_mode;
    const uint32_t* given;     // position-order bits when GIVEN
    int32_t sample;            // index of the instance in the context
    float xslope;              // 2 beta / sqrt(N): thr[x] ~ 2^32 exp(-xslope x)
    // real couplings (sg_skg.hip): Jw, H, thr unused
    const float* Jf;           // [n][skg_pitch(n)], zero past n
    float* Jd;                 // [ceil(n / 64)][64][64] strict upper triangles of the diagonal tiles
    double* Hd;                // [n] local fields between launches
    double beta;               // 1 / T
};

// SK instance (sample) for the exact field recompute: all its chains.
struct SkSample {
    const uint64_t* Jw;
    int32_t n;
    int32_t nch;
    int32_t chain0;            // index of its first chain in the chain array
    int32_t pad_;
    const float* Jf;           // real couplings, or null
};

struct MeasureChain {
    const uint32_t* snap;      // [K][words_n]
    int32_t words_n;
    int32_t n;
};

// ---- launchers (return hipError_t) ----
hipError_t vb_init(const VbUnit* units, int n_units, int threads, size_t lds_bytes, hipStream_t s);
// One-time kernel attributes (large dynamic LDS); call before launching or
// capturing VB sweeps.
hipError_t vb_prepare();
// t0p: device counter of sweeps done, read by the kernel; vb_advance adds
// n_sweeps to it on the stream (after every launch group of a chunk).
hipError_t vb_sweep(const VbUnit* units, int n_units, int threads, size_t lds_bytes, const int64_t* t0p,
                    int32_t n_sweeps, int64_t t_max, hipStream_t s);
// also zeroes the n_bar barrier words of split units for the next launch
hipError_t vb_advance(int64_t* t, int32_t n_sweeps, uint32_t* bars, int n_bar, hipStream_t s);
// LDS a unit needs for a launch with `threads` lanes per workgroup, and the
// extra LDS that keeps its whole adjacency resident.
size_t vb_lds_bytes(int32_t n, int32_t rpad, int32_t nch, int threads, bool cpl = false);
// Adjacency entries (position | (J < 0) << 31) in the form a unit with a
// complemented copy of its spin words reads: the LDS byte address of the
// neighbour's word, of its complement when J < 0, above 5 bits of in-word
// shift; `pad` entries of position 0 follow the m entries.
void vb_cpl_entries(const uint32_t* ent, size_t m, size_t pad, int32_t rpad, int32_t n, uint32_t* out);
size_t vb_resident_bytes(int32_t n, int32_t m2, int32_t ncls);

// Multispin units (sg_vbm.hip).
size_t vbm_lds_bytes(int32_t n, int threads);
hipError_t vbm_init(const VbmUnit* units, int n_units, hipStream_t s);
hipError_t vbm_prepare();
hipError_t vbm_sweep(const VbmUnit* units, int n_units, int threads, size_t lds_bytes, const int64_t* t0p,
                     int32_t n_sweeps, int64_t t_max, hipStream_t s);
// bond sums of the snapshots k_first .. k_done - 1 of every chain of every
// unit: out[chain][k], chain ids [unit][64]
hipError_t vbm_bond(const VbmUnit* units, int n_units, int k_first, int k_done, long long* out,
                    const int32_t* chain_ids, int k_cap, hipStream_t s);

// err_flag bit 0: recompute mismatch; bit 1: the sweep pipeline stalled.
hipError_t sk_init(const SkChain* chains, int n_chains, int threads, hipStream_t s);
hipError_t sk_recompute(const SkSample* samples, int n_samples, const SkChain* chains,
                        int max_n, int max_nch, int check, int* err_flag, hipStream_t s);
hipError_t sk_bond(const SkSample* samples, int n_samples, const SkChain* chains, int max_n,
                   int k_done, int k_cap, long long* out, hipStream_t s);
hipError_t sk_sweep(const SkChain* chains, int n_chains, int max_n, size_t lds_bytes, int64_t t0,
                    int32_t n_sweeps, int64_t t_max, int* err_flag, hipStream_t s);
size_t sk_lds_bytes(int32_t n);
// Bytes that the sweep kernel may read (and not use) past a matrix Jw: readable
// memory of the context follows each.
constexpr size_t kSkOverread = (size_t)12 * 48 * 1024;

// SK with real couplings (sg_skg.hip): sweeps, direct field recomputation
// (with `check`, error bit 0 when a field drifted by more than 1e-9 (1 + |h|))
// and bond sums of the snapshots (partials `part` of samples x max_nch x k_cap x
// skg_row_blocks(max_n) doubles; out[chain][k]).
int skg_row_blocks(int32_t n);
size_t skg_lds_bytes(int32_t n);
hipError_t skg_diag(const SkSample* samples, int n_samples, const SkChain* chains, int max_n, hipStream_t s);
hipError_t skg_sweep(const SkChain* chains, int n_chains, int max_n, size_t lds_bytes, int64_t t0, int32_t n_sweeps,
                     int64_t t_max, int* err_flag, hipStream_t s);
hipError_t skg_recompute(const SkSample* samples, int n_samples, const SkChain* chains, int max_n, int check,
                         int* err_flag, hipStream_t s);
hipError_t skg_bond(const SkSample* samples, int n_samples, const SkChain* chains, int max_n, int max_nch,
                    int k_done, int k_cap, double* part, double* out, hipStream_t s);

// bond sums of the snapshots k_first .. k_done - 1 of every chain of the units:
// bond_out[chain][k] (the other times are left as they are; bond_out has n_chains
// rows, and those of other chains become 0 at these times)
hipError_t vb_bond(const VbUnit* units, int n_units, int n_chains, int max_n, int k_first, int k_done, long long* bond_out,
                   const int32_t* unit_chain_ids, int k_cap, int threads, size_t lds_bytes,
                   hipStream_t s);
// Counts of unequal spins over every pair of a chain's first k_done snapshots
// (gram_cnt[chain][l (l - 1) / 2 + k], k < l; chains hold k_cap (k_cap - 1) / 2)
// and of two replicas at each of those times (ovl_cnt[pair][k_cap]).  The counts
// are zero before; observe_expand and observe_pack clear what they read.
hipError_t observe(const MeasureChain* chains, int n_chains, int count, int R, int k_done, int k_cap, int max_words,
                   uint32_t* gram_cnt, uint32_t* ovl_cnt, hipStream_t s);
// The counts as Gram matrices [chain][k_cap][k_cap] and overlaps [pair][k_cap].
hipError_t observe_expand(const MeasureChain* chains, int n_chains, int n_pairs, int R, int k_done, int k_cap,
                          uint32_t* gram_cnt, uint32_t* ovl_cnt, long long* gram, long long* ovl, hipStream_t s);
// Copies the destination words w0 .. w1 - 1 of the segments to mapped host memory (w0
// to dst[0]) and clears those that ask for it (dst null: only clears)
hipError_t observe_pack(const PackList& list, uint32_t* dst, uint64_t w0, uint64_t w1, hipStream_t s);
hipError_t zero_i64(long long* p, size_t n, hipStream_t s);
// Device address of the fixed staging array (kMeasureScratchElems int64) on
// the current device; looked up once per device.
hipError_t measure_scratch(long long** ptr);

}  // namespace sg
