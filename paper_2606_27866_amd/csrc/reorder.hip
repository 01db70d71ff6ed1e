// One-time channel ranking and reorder (FlexMoE Sec. 3.1, Eq. 3).
//   rank_kernel: position of channel c in the stable descending order of the
//     scores = #{j : (s_j, j) precedes (s_c, c)}, with NaN after every
//     number.  The order is total, so the positions form a permutation and
//     perm[e][position] = c.
//   gather_rows_kernel: W~_gate[e][c] = W_gate[e][perm[e][c]] (and up).
//   gather_cols_lds_kernel: W~_down[e][n][c] = W_down[e][n][perm[e][c]].
// The copies are bound by memory; what they took on the Qwen1.5-MoE shape
// (60 experts, 1408 channels, hidden size 2048, bf16) stands at each kernel.
#include "kernels.h"

namespace flexmoe {

// A key whose unsigned order is the scores' order: a larger score has a
// larger key, -0 and +0 share one, NaN has the smallest (0).  No key is
// 0xffffffff.
__device__ __forceinline__ uint32_t score_key(float v) {
    const uint32_t u = __float_as_uint(v == 0.f ? 0.f : v);
    if (__builtin_isnan(v)) return 0u;
    return u >> 31 ? ~u : u | 0x80000000u;
}

// One thread per channel c counts the channels before it: those with a larger
// key, and the lower-numbered ones with an equal key.  For j < c that is
// key_j >= key_c, for j > c key_j >= key_c + 1, so outside the workgroup's own
// 256 channels a pair costs one compare and one add against a fixed threshold
// (160 -> 25 us; the scores were compared as floats with ties and NaN
// decided per pair).
constexpr int kRankThreads = 256;
__global__ __launch_bounds__(kRankThreads) void rank_kernel(const float* __restrict__ scores, int I,
                                                            int32_t* __restrict__ perm) {
    constexpr int CH = 2048;
    static_assert(CH % kRankThreads == 0, "a workgroup's channels lie in one chunk");
    __shared__ __attribute__((aligned(16))) uint32_t sk[CH];
    const int e = blockIdx.y;
    const int c0 = blockIdx.x * kRankThreads, c = c0 + threadIdx.x;
    const float* s = scores + (size_t)e * I;
    const uint32_t key = c < I ? score_key(s[c]) : 0u;
    int rank = 0;
    // pairs with keys [lo, hi) of the chunk (multiples of 4) at threshold t
    auto count = [&](int lo, int hi, uint32_t t) {
#pragma unroll 4
        for (int j = lo; j < hi; j += 4) {
            const u32x4 k = *reinterpret_cast<const u32x4*>(sk + j);
#pragma unroll
            for (int q = 0; q < 4; ++q) rank += k[q] >= t ? 1 : 0;
        }
    };
    for (int j0 = 0; j0 < I; j0 += CH) {
        const int n = min(CH, I - j0);
        __syncthreads();
        // keys past the end are 0: below every threshold t >= 1, and never
        // compared with a lower one (they are past every channel)
        for (int j = threadIdx.x; j < CH; j += kRankThreads) sk[j] = j < n ? score_key(s[j0 + j]) : 0u;
        __syncthreads();
        const int own = c0 - j0;  // this workgroup's channels in the chunk
        const int n4 = (n + 3) & ~3;
        if (own >= n) {
            count(0, n4, key);
        } else if (own + kRankThreads <= 0) {
            count(0, n4, key + 1);
        } else {
            count(0, own, key);
            const int end = min(own + kRankThreads, n);
            const int mine = own + threadIdx.x;
#pragma unroll 4
            for (int j = own; j < end; ++j) rank += sk[j] >= key + (j < mine ? 0u : 1u) ? 1 : 0;
            count(min(own + kRankThreads, n4), n4, key + 1);
        }
    }
    if (c < I) perm[(size_t)e * I + rank] = c;
}

// 16 bytes that are read once and written once
__device__ __forceinline__ void copy16(void* dst, const void* src) {
    __builtin_nontemporal_store(__builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src)),
                                reinterpret_cast<u32x4*>(dst));
}

// one block per (expert, ranked channel); rows are copied in 16-byte pieces
// with the non-temporal hint (247 -> 227 us, 6.1 TB/s of reads and writes)
__global__ __launch_bounds__(128) void gather_rows_kernel(const uint8_t* __restrict__ wg,
                                                          const uint8_t* __restrict__ wu,
                                                          uint8_t* __restrict__ wg_r,
                                                          uint8_t* __restrict__ wu_r,
                                                          const int32_t* __restrict__ perm, int I,
                                                          size_t row_bytes) {
    const size_t e = blockIdx.y, c = blockIdx.x;
    const size_t src = (e * I + (size_t)perm[e * I + c]) * row_bytes;
    const size_t dst = (e * I + c) * row_bytes;
    for (size_t b = threadIdx.x * 16; b < row_bytes; b += blockDim.x * 16) {
        copy16(wg_r + dst + b, wg + src + b);
        copy16(wu_r + dst + b, wu + src + b);
    }
}

// Columns of W_down permuted: `rows` rows of one expert go through LDS, read
// and written in 16-byte pieces; a thread takes the 8 positions of a ranked
// chunk once and gathers them for every row (350 -> 119 us: gathering
// 2-byte elements from memory kept the address units busy, not the memory).
template <typename T>
__global__ __launch_bounds__(256) void gather_cols_lds_kernel(const T* __restrict__ wd, T* __restrict__ wd_r,
                                                              const int32_t* __restrict__ perm, int I, int d,
                                                              int rows) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int VEC = 16 / sizeof(T);
    T* row = reinterpret_cast<T*>(smem);
    const size_t e = blockIdx.y;
    const int n0 = blockIdx.x * rows, nr = min(rows, d - n0);
    const size_t base = (e * d + n0) * (size_t)I;  // the rows are contiguous
    const int chunks = nr * (I / VEC);             // I % 8 == 0
    for (int k = threadIdx.x; k < chunks; k += 256)
        reinterpret_cast<u32x4*>(row)[k] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wd + base) + k);
    __syncthreads();
    const int32_t* pe = perm + e * I;
    for (int k = threadIdx.x; k < I / 8; k += 256) {
        int p[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) p[j] = pe[k * 8 + j];
        for (int r = 0; r < nr; ++r) {
            T v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = row[r * I + p[j]];
#pragma unroll
            for (int q = 0; q < 8 / VEC; ++q)
                __builtin_nontemporal_store(
                    reinterpret_cast<const u32x4*>(v)[q],
                    reinterpret_cast<u32x4*>(wd_r + base + (size_t)r * I + k * 8 + q * VEC));
        }
    }
}

// The same without LDS and without vector accesses: rows longer than
// kColsLds, or down matrices that are not 16-byte aligned.
constexpr int kColsLds = 64 * 1024;      // LDS a workgroup gets without asking for more
constexpr int kColsTarget = 24 * 1024;   // six workgroups per compute unit
constexpr int kColsRows = 8;             // rows that share a thread's permutation entries
template <typename T>
__global__ __launch_bounds__(256) void gather_cols_kernel(const T* __restrict__ wd, T* __restrict__ wd_r,
                                                          const int32_t* __restrict__ perm, int I, int d) {
    const size_t e = blockIdx.y, n = blockIdx.x;
    const T* src = wd + (e * d + n) * (size_t)I;
    T* dst = wd_r + (e * d + n) * (size_t)I;
    const int32_t* pe = perm + e * I;
    for (int c = threadIdx.x; c < I; c += blockDim.x) dst[c] = src[pe[c]];
}

template <typename T>
static hipError_t launch_gather_cols(const T* wd, T* wd_r, const int32_t* perm, int E, int I, int d, hipStream_t s) {
    const size_t row = (size_t)I * sizeof(T);
    if (row > kColsLds || (((uintptr_t)wd | (uintptr_t)wd_r) & 15)) {
        gather_cols_kernel<T><<<dim3(d, E), 256, 0, s>>>(wd, wd_r, perm, I, d);
        return hipGetLastError();
    }
    const int rows = max(1, min(kColsRows, (int)(kColsTarget / row)));
    gather_cols_lds_kernel<T><<<dim3(ceil_div(d, rows), E), 256, rows * row, s>>>(wd, wd_r, perm, I, d, rows);
    return hipGetLastError();
}

hipError_t launch_rank_reorder(const float* scores, const void* wg, const void* wu, const void* wd,
                               void* wg_r, void* wu_r, void* wd_r, int32_t* perm, int E, int I,
                               int d, int esize, hipStream_t s) {
    rank_kernel<<<dim3(ceil_div(I, kRankThreads), E), kRankThreads, 0, s>>>(scores, I, perm);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    gather_rows_kernel<<<dim3(I, E), 128, 0, s>>>((const uint8_t*)wg, (const uint8_t*)wu,
                                                   (uint8_t*)wg_r, (uint8_t*)wu_r, perm, I,
                                                   (size_t)d * esize);
    err = hipGetLastError();
    if (err != hipSuccess) return err;
    return esize == 2 ? launch_gather_cols((const bf16_t*)wd, (bf16_t*)wd_r, perm, E, I, d, s)
                      : launch_gather_cols((const float*)wd, (float*)wd_r, perm, E, I, d, s);
}

}  // namespace flexmoe
