// Observables at the grid times, from the device-resident snapshots.
//
//  * Gram matrices G[k][l] = sum_i s_i(t_k) s_i(t_l) per chain (the two-time
//    correlation C = G / N of the introduction and SI Eq. formula1) and
//    two-clone overlaps Q = sum_i s^a_i s^b_i: N - 2 popcount(x xor y) over the
//    packed spins, for every pair of rows of a set (a chain's snapshots, or the
//    replicas' snapshots of one time).
//  * VB bond sums B = sum_{(uv) in E} J_uv s_u s_v (energy -B, Eq. 3), one
//    pass over the unit's adjacency per snapshot time.
#include "sg_internal.h"

#include <mutex>

// Staging of sg_measure_noalloc (bond sums, overlaps, Gram matrices before
// they are copied to the caller's host arrays): a fixed device array instead
// of memory allocated by the library.  Each device holds its own copy until
// the process ends.  In host code the name stands for a host-side shadow, so
// the kernels get the device address from measure_scratch() instead.
static __device__ __align__(256) long long scratch[sg::kMeasureScratchElems];

namespace sg {
namespace {

// Sum over the 256 threads' pair counts: grid = the Gram sets' tiles (chains x
// g_tiles), then the overlap sets' tiles (instances x times x o_tiles).  A block
// stages one tile of a set's rows in LDS and counts popcount(x xor y) for every
// pair of rows.  A thread takes a 2 x 2 block of pairs (four 16-byte LDS reads
// for 4 pairs of 128 spins) and one of `parts` interleaved column sets of the
// tile, so that few rows still occupy the block; parts are added in LDS.  One
// tile per set: plain stores; more: the counts are added to `gram` / `ovl`,
// which hold zeros between measurements.
//
// With one bit per spin a pair of 32 spins costs an XOR and a count; on the
// matrix cores the spins would have to be spread to bytes first, at 20
// instructions per 16 spins of each row (below about 200 rows the pairs are
// cheaper).  Measured, Gram matrices and overlaps together: 16384 chains of 4096
// spins, 12 times, 28 pairs an instance 124 us (1410 + 180 us as one block per
// pair and time and int8 products, one wavefront per 8192 spins); 1536 chains of
// 65536 spins, 10 times, one pair 91 us (300).  Bound by staging: 2 loads in
// flight a lane and a barrier before the counting.
struct ObsPlan {
    int32_t n_chains, R, kd;
    int32_t g_tiles, g_words;   // tiles per chain, words per tile (a multiple of 64)
    int32_t o_tiles, o_words;
    int32_t g_stride, o_stride; // entries per chain (all pairs of K rows), per pair of replicas (K)
};

__global__ void __launch_bounds__(256) observe_kernel(const MeasureChain* __restrict__ chains, ObsPlan p,
                                                      uint32_t* __restrict__ gram, uint32_t* __restrict__ ovl)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t osm[];
    __shared__ uint32_t cnt[kMaxGrid * (kMaxGrid - 1) / 2];
    const int tid = threadIdx.x;
    const int32_t g_blocks = p.n_chains * p.g_tiles;
    const bool is_gram = (int32_t)blockIdx.x < g_blocks;
    int32_t id, tile, k = 0, chain;
    if (is_gram) {
        id = (int32_t)blockIdx.x / p.g_tiles;
        tile = (int32_t)blockIdx.x - id * p.g_tiles;
        chain = id;
    } else {
        const int32_t b = (int32_t)blockIdx.x - g_blocks;
        const int32_t set = b / p.o_tiles;
        tile = b - set * p.o_tiles;
        id = set / p.kd;
        k = set - id * p.kd;
        chain = id * p.R;
    }
    const int32_t wn = chains[chain].words_n, n = chains[chain].n;
    const int32_t T = is_gram ? p.g_words : p.o_words, rows = is_gram ? p.kd : p.R;
    const int32_t w0 = tile * T;
    if (w0 >= wn) return;
    const int32_t nw = min(T, wn - w0), c4 = (nw + 3) >> 2, ld = T + 4;
    const int32_t last = w0 + nw == wn && (n & 31) ? nw - 1 : -1;   // the word that ends inside
    const uint32_t keep = last >= 0 ? (1u << (n & 31)) - 1u : ~0u;
    // stage the rows; words past the tile are zero in every row
    for (int32_t r = 0; r < rows; ++r) {
        const uint32_t* src = (is_gram ? chains[chain].snap + (int64_t)r * wn : chains[chain + r].snap + (int64_t)k * wn) + w0;
        uint32_t* dst = osm + r * ld;
        if (((uintptr_t)src & 15) == 0) {
            for (int32_t j = tid; j < c4; j += 256) {
                uint4 v = make_uint4(0u, 0u, 0u, 0u);
                const int32_t w = 4 * j;
                if (w + 4 <= nw) {
                    v = *(const uint4*)(src + w);
                } else {
                    v.x = src[w];
                    if (w + 1 < nw) v.y = src[w + 1];
                    if (w + 2 < nw) v.z = src[w + 2];
                }
                *(uint4*)(dst + w) = v;
            }
        } else {
            for (int32_t w = tid; w < 4 * c4; w += 256) dst[w] = w < nw ? src[w] : 0u;
        }
    }
    const int32_t np = rows * (rows - 1) / 2;
    for (int32_t i = tid; i < np; i += 256) cnt[i] = 0u;
    __syncthreads();
    const int32_t g = (rows + 1) >> 1, nb = g * (g + 1) / 2, parts = max(1, 256 / nb);
    if (tid < nb * parts) {
        const int32_t part = tid / nb, blk = tid - part * nb;
        int32_t J = 0, base = 0;
        while (base + J + 1 <= blk) {
            base += J + 1;
            ++J;
        }
        const int32_t I = blk - base;   // I <= J
        const int32_t a0 = 2 * I, a1 = min(2 * I + 1, rows - 1), b0 = 2 * J, b1 = min(2 * J + 1, rows - 1);
        const uint32_t *pa0 = osm + a0 * ld, *pa1 = osm + a1 * ld, *pb0 = osm + b0 * ld, *pb1 = osm + b1 * ld;
        uint32_t s00 = 0u, s01 = 0u, s10 = 0u, s11 = 0u;
        const int32_t last4 = last >= 0 ? last >> 2 : -1;
        for (int32_t j = part; j < c4; j += parts) {
            uint4 x0 = *(const uint4*)(pa0 + 4 * j), x1 = *(const uint4*)(pa1 + 4 * j);
            uint4 y0 = *(const uint4*)(pb0 + 4 * j), y1 = *(const uint4*)(pb1 + 4 * j);
            if (j == last4) {
                auto mask = [&](uint4& v) {
                    uint32_t* e = &v.x;
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (4 * j + i == last) e[i] &= keep;
                };
                mask(x0);
                mask(x1);
                mask(y0);
                mask(y1);
            }
            auto add = [](uint32_t& s, const uint4& x, const uint4& y) {
                s += __popc(x.x ^ y.x) + __popc(x.y ^ y.y) + __popc(x.z ^ y.z) + __popc(x.w ^ y.w);
            };
            add(s00, x0, y0);
            add(s01, x0, y1);
            add(s10, x1, y0);
            add(s11, x1, y1);
        }
        // (k < l at l (l - 1) / 2 + k; a doubled last row or a pair of a diagonal block's mirror is dropped)
        auto put = [&](int32_t a, int32_t b, uint32_t v) {
            if (a < b && v != 0u) atomicAdd(&cnt[b * (b - 1) / 2 + a], v);
        };
        put(a0, b0, s00);
        if (2 * J + 1 < rows) put(a0, b1, s01);
        if (2 * I + 1 < rows) {
            put(a1, b0, s10);
            if (2 * J + 1 < rows) put(a1, b1, s11);
        }
    }
    __syncthreads();
    for (int32_t i = tid; i < np; i += 256) {
        uint32_t* o;
        if (is_gram) {
            o = gram + (int64_t)id * p.g_stride + i;
        } else {
            // replicas (a, b) in lexicographic order
            int32_t b = 1;
            while ((b + 1) * b / 2 <= i) ++b;
            const int32_t a = i - b * (b - 1) / 2;
            const int32_t q = a * p.R - a * (a + 1) / 2 + (b - a - 1);
            o = ovl + ((int64_t)id * np + q) * p.o_stride + k;
        }
        const uint32_t v = cnt[i];
        if ((is_gram ? p.g_tiles : p.o_tiles) == 1)
            *o = v;
        else if (v != 0u)
            atomicAdd(o, v);
    }
}

// Counts to the observables' own form, in device memory: Gram matrices of K x K
// and overlaps of K entries a pair, zero past the k_done times reached; the
// counts are cleared.
__global__ void __launch_bounds__(256) expand_kernel(const MeasureChain* __restrict__ chains, int32_t n_chains,
                                                     int32_t n_pairs, int32_t per_inst, int32_t R, int32_t kd,
                                                     int32_t K, uint32_t* __restrict__ gram_cnt,
                                                     uint32_t* __restrict__ ovl_cnt, long long* __restrict__ gram,
                                                     long long* __restrict__ ovl)
{
    const int32_t np = K * (K - 1) / 2;
    const int64_t step = (int64_t)gridDim.x * blockDim.x, i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = i0; i < (int64_t)n_chains * K * K; i += step) {
        const int64_t ch = i / (K * K);
        const int32_t e = (int32_t)(i - ch * (K * K)), l = e / K, k = e - l * K;
        if (k > l) continue;
        long long v = 0;
        if (l < kd) {
            v = chains[ch].n;
            if (k < l) {
                uint32_t* p = gram_cnt + ch * np + l * (l - 1) / 2 + k;
                v -= 2LL * *p;
                *p = 0u;
            }
        }
        gram[ch * (K * K) + l * K + k] = v;
        gram[ch * (K * K) + k * K + l] = v;
    }
    for (int64_t i = i0; i < (int64_t)n_pairs * K; i += step) {
        const int64_t q = i / K;
        const int32_t k = (int32_t)(i - q * K);
        ovl[i] = k < kd ? (long long)chains[q / per_inst * R].n - 2LL * ovl_cnt[i] : 0;
        ovl_cnt[i] = 0u;
    }
}

// Copies the destination words w0 .. w1 - 1 of a measurement's segments, one segment
// after another, to mapped host memory (4 bytes a lane: 53 GB/s, the link's rate, as a
// DMA copy of one piece; without a destination: nothing), and clears those that hold
// counts.
__global__ void __launch_bounds__(256) pack_kernel(PackList L, uint32_t* __restrict__ dst, uint64_t w0, uint64_t w1)
{
    const uint64_t step = (uint64_t)gridDim.x * blockDim.x, i0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int s = 0; s < L.n; ++s) {
        const PackSeg g = L.seg[s];
        const uint64_t a = max(w0, g.dst), e = min(w1, g.dst + pack_words(g));
        for (uint64_t w = a + i0; w < e; w += step) {
            uint32_t* p = g.src + pack_from(g, w - g.dst);
            if (dst) dst[w - w0] = *p;
            if (g.clear) *p = 0u;
        }
    }
}

// Positions of a unit that one workgroup of vb_bond_kernel sums over.
constexpr int kBondSlice = 32768;

// grid = (units, times, slices of kBondSlice positions).  Snapshot bits of the
// unit's chains are staged in LDS chain-major; the workgroup visits the adjacency of
// its slice, each edge from its lower end, and adds its sums to `out` (zero before).
// A graph's slices each stage all its spins (128 KB for 2^20 spins and one chain, from
// L2) so that one large graph does not leave the chip to a single workgroup.
// Measured, one new time: two chains of 985767 spins 250 us (1520 with one workgroup
// a unit; slices of 16384 290, 8192 390), 512 chains of 2^10 to 2^20 spins 470 (2250).
// Bound by staging and by the gathers' latency at one workgroup a CU.
__global__ void __launch_bounds__(1024) vb_bond_kernel(const VbUnit* __restrict__ units,
                                                       const int32_t* __restrict__ chain_ids,
                                                       int k_first, int k_cap, long long* __restrict__ out)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t bsm[];
    const VbUnit* up = units + blockIdx.x;
    if (up->member != 0) return;   // a split unit is measured once
    const int k = k_first + (int)blockIdx.y;
    const int32_t n = up->n, wn = up->words_n, nch = up->nch;
    const int32_t p0 = (int32_t)blockIdx.z * kBondSlice, p1 = min(n, p0 + kBondSlice);
    if (p0 >= n) return;
    long long* red = (long long*)(bsm + ((nch * wn + 1) & ~1));
    const int bd = (int)blockDim.x;
    for (int c = 0; c < nch; ++c) {
        const uint32_t* src = up->snap[c] + (int64_t)k * wn;
        uint32_t* dst = bsm + c * wn;
        int32_t w = (int32_t)threadIdx.x;
        for (; w + 7 * bd < wn; w += 8 * bd) {
            uint32_t v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = src[w + j * bd];
#pragma unroll
            for (int j = 0; j < 8; ++j) dst[w + j * bd] = v[j];
        }
        for (; w < wn; w += bd) dst[w] = src[w];
    }
    if (threadIdx.x < kVbMaxChains) red[threadIdx.x] = 0;
    __syncthreads();
    int32_t sum[kVbMaxChains];
#pragma unroll
    for (int c = 0; c < kVbMaxChains; ++c) sum[c] = 0;
    const int32_t* __restrict__ row = up->row;
    const uint32_t* __restrict__ ent = up->ent;
    // four positions of a thread at a time, four entries of each (the adjacency is
    // followed by kVbEntPad zeros): their loads are in flight together
    for (int32_t p = p0 + (int32_t)threadIdx.x; p < p1; p += 4 * bd) {
        int32_t e0[4], e1[4];
        uint32_t own[4];   // bit c: chain c's spin
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int32_t pj = p + j * bd;
            e0[j] = pj < p1 ? row[pj] : 0;
            e1[j] = pj < p1 ? row[pj + 1] : 0;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int32_t pj = min(p + j * bd, n - 1);
            own[j] = 0u;
#pragma unroll
            for (int c = 0; c < kVbMaxChains; ++c)
                if (c < nch) own[j] |= ((bsm[c * wn + (pj >> 5)] >> (pj & 31)) & 1u) << c;
        }
        while (e0[0] < e1[0] || e0[1] < e1[1] || e0[2] < e1[2] || e0[3] < e1[3]) {
            uint32_t en[4][4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) en[j][i] = ent[min(e0[j], e1[j]) + i];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int32_t q = (int32_t)(en[j][i] & 0x7fffffffu);
                    if (e0[j] + i >= e1[j] || q < p + j * bd) continue;
                    const uint32_t neg = en[j][i] >> 31;
#pragma unroll
                    for (int c = 0; c < kVbMaxChains; ++c) {
                        if (c >= nch) break;
                        const uint32_t bq = bsm[c * wn + (q >> 5)] >> (q & 31);
                        sum[c] += 1 - 2 * (int32_t)(((own[j] >> c) ^ bq ^ neg) & 1u);
                    }
                }
                e0[j] += 4;
            }
        }
    }
#pragma unroll
    for (int c = 0; c < kVbMaxChains; ++c)
        if (c < nch && sum[c] != 0)
            atomicAdd((unsigned long long*)&red[c], (unsigned long long)(long long)sum[c]);
    __syncthreads();
    if (threadIdx.x < nch && red[threadIdx.x] != 0)
        atomicAdd((unsigned long long*)&out[(int64_t)chain_ids[blockIdx.x * kVbMaxChains + threadIdx.x] * k_cap + k],
                  (unsigned long long)red[threadIdx.x]);
}

// out[i][k_first .. k_done) = 0 for every row of k_cap.
__global__ void zero_columns_kernel(long long* out, int64_t rows, int k_first, int k_done, int k_cap)
{
    const int w = k_done - k_first;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < rows * w; i += (int64_t)gridDim.x * blockDim.x)
        out[i / w * k_cap + k_first + i % w] = 0;
}

__global__ void zero_kernel(long long* p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

}  // namespace

hipError_t zero_i64(long long* p, size_t n, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    const int blocks = (int)std::min<size_t>(1024, (n + 255) / 256);
    hipLaunchKernelGGL(zero_kernel, dim3(blocks), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t measure_scratch(long long** ptr)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static long long* addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        // once per device, with that device current: its copy's address
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = static_cast<long long*>(p);
    }
    *ptr = addr[dev];
    return hipSuccess;
}

hipError_t observe(const MeasureChain* chains, int n_chains, int count, int R, int k_done, int k_cap, int max_words,
                   uint32_t* gram_cnt, uint32_t* ovl_cnt, hipStream_t s)
{
    if (n_chains <= 0 || k_done <= 0) return hipSuccess;
    // tiles of at most 32 KB
    constexpr int kTile = 8192;
    auto words = [&](int rows) { return std::min((max_words + 63) & ~63, (kTile / rows) & ~63); };
    ObsPlan p;
    p.n_chains = k_done > 1 ? n_chains : 0;
    p.R = R;
    p.kd = k_done;
    p.g_words = words(k_done);
    p.g_tiles = (max_words + p.g_words - 1) / p.g_words;
    p.o_words = words(R);
    p.o_tiles = (max_words + p.o_words - 1) / p.o_words;
    p.g_stride = k_cap * (k_cap - 1) / 2;
    p.o_stride = k_cap;
    const int64_t blocks = (int64_t)p.n_chains * p.g_tiles + (R > 1 ? (int64_t)count * k_done * p.o_tiles : 0);
    if (blocks <= 0) return hipSuccess;
    if (blocks > 0x7fffffff) return hipErrorInvalidConfiguration;
    const size_t lds = 4 * (size_t)std::max(k_done > 1 ? k_done * (p.g_words + 4) : 0, R > 1 ? R * (p.o_words + 4) : 0);
    hipLaunchKernelGGL(observe_kernel, dim3((unsigned)blocks), dim3(256), lds, s, chains, p, gram_cnt, ovl_cnt);
    return hipGetLastError();
}

hipError_t observe_expand(const MeasureChain* chains, int n_chains, int n_pairs, int R, int k_done, int k_cap,
                          uint32_t* gram_cnt, uint32_t* ovl_cnt, long long* gram, long long* ovl, hipStream_t s)
{
    const int64_t work = std::max((int64_t)n_chains * k_cap * k_cap, (int64_t)n_pairs * k_cap);
    const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>(2048, (work + 255) / 256));
    hipLaunchKernelGGL(expand_kernel, dim3(blocks), dim3(256), 0, s, chains, n_chains, n_pairs,
                       std::max(1, R * (R - 1) / 2), R, k_done, k_cap, gram_cnt, ovl_cnt, gram, ovl);
    return hipGetLastError();
}

hipError_t observe_pack(const PackList& list, uint32_t* dst, uint64_t w0, uint64_t w1, hipStream_t s)
{
    uint64_t most = 0;
    for (int i = 0; i < list.n; ++i) most = std::max(most, std::min(w1 - w0, pack_words(list.seg[i])));
    const int blocks = (int)std::max<uint64_t>(1, std::min<uint64_t>(512, (most + 255) / 256));
    hipLaunchKernelGGL(pack_kernel, dim3(blocks), dim3(256), 0, s, list, dst, w0, w1);
    return hipGetLastError();
}

hipError_t vb_bond(const VbUnit* units, int n_units, int n_chains, int max_n, int k_first, int k_done, long long* bond_out,
                   const int32_t* unit_chain_ids, int k_cap, int threads, size_t lds_bytes,
                   hipStream_t s)
{
    if (n_units <= 0 || k_done <= k_first) return hipSuccess;
    // set once (thread-safe initialisation of a local static)
    static const hipError_t attr = hipFuncSetAttribute((const void*)vb_bond_kernel,
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return attr;
    const int64_t cells = (int64_t)n_chains * (k_done - k_first);
    hipLaunchKernelGGL(zero_columns_kernel, dim3((unsigned)std::min<int64_t>(1024, (cells + 255) / 256)), dim3(256), 0, s,
                       bond_out, (int64_t)n_chains, k_first, k_done, k_cap);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(vb_bond_kernel, dim3(n_units, k_done - k_first, (max_n + kBondSlice - 1) / kBondSlice), dim3(threads),
                       lds_bytes, s, units, unit_chain_ids, k_first, k_cap, bond_out);
    return hipGetLastError();
}

}  // namespace sg
