// Offline clipping (FlexMoE Sec. 4.4, Table 2): the subnetwork of one budget
// exported as a standalone set of compact weights, which the same GEMM
// kernels read through the clipped layout of RoutedWeights (kernels.h).
//
// Expert e keeps its first k_e ranked channels, padded to kp_e =
// packed_width(k_e) (a multiple of 8, so every packed row is 16-byte
// aligned):
//   gate/up  [kp_e][d]  rows c < k_e copied from the ranked rows, the rest 0
//   down     [d][kp_e]  columns c < k_e copied from the ranked columns, the rest 0
// and the experts' blocks follow one another in expert order, expert e
// starting at packed channel ch0_e = sum_{e' < e} kp_e' (element ch0_e * d of
// every packed matrix).  The padding is never multiplied into a result: the
// gate/up GEMM computes channels below k_e only, and the down GEMM's zero H
// columns meet the zero padding.
#include "kernels.h"

namespace flexmoe {

namespace {
struct ExportArgs {
    KeepArgs keep;  // k_e
    KeepArgs ch0;   // first packed channel of each expert
};

// One expert (blockIdx.y) and one matrix (blockIdx.z: gate, up, down), a
// grid-stride walk over its packed block in 16-byte chunks (VEC elements).
// Bound by memory: each kept byte is read and written once (220 -> 194 us, 5.3 TB/s,
// for half of the channels of the Qwen1.5-MoE shape: the down columns were
// read element by element, and every chunk divided 64-bit indexes).
template <typename T>
__global__ __launch_bounds__(256) void export_clipped_kernel(ExportArgs a, const T* __restrict__ wg_r,
                                                             const T* __restrict__ wu_r,
                                                             const T* __restrict__ wd_r, T* __restrict__ wg_c,
                                                             T* __restrict__ wu_c, T* __restrict__ wd_c, int I,
                                                             int d) {
    constexpr int VEC = 16 / sizeof(T);
    const int e = blockIdx.y;
    const int k = a.keep.v[e], kp = packed_width(k);
    const size_t src = (size_t)e * I * d;                // ranked block of expert e
    const size_t dst = (size_t)a.ch0.v[e] * d;           // packed block of expert e
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const size_t first = (size_t)blockIdx.x * blockDim.x + threadIdx.x, step = (size_t)gridDim.x * blockDim.x;
    if (blockIdx.z < 2) {
        // gate/up: the packed rows are the first k ranked rows, then zeros
        const u32x4* w = reinterpret_cast<const u32x4*>((blockIdx.z ? wu_r : wg_r) + src);
        u32x4* out = reinterpret_cast<u32x4*>((blockIdx.z ? wu_c : wg_c) + dst);
        const size_t kept = (size_t)k * d / VEC, n = (size_t)kp * d / VEC;  // d % 8 == 0
        for (size_t i = first; i < n; i += step)
            __builtin_nontemporal_store(i < kept ? __builtin_nontemporal_load(w + i) : zero, out + i);
    } else {
        // down: packed element (n, c) = ranked (n, c) for c < k, else 0; rows
        // of both start on 16-byte boundaries (I % 8 == 0, kp % 8 == 0)
        const unsigned kc = kp / VEC;
        const size_t n = (size_t)d * kc;
        for (size_t i = first; i < n; i += step) {
            // row and chunk of the row: in 32 bits where the block allows it
            const size_t r = n >> 32 ? i / kc : (unsigned)i / kc;
            const int c = (int)(i - r * kc) * VEC;
            union {
                u32x4 v;
                T t[VEC];
            } x;
            x.v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(wd_r + src + r * I + c));
            if (c + VEC > k)
#pragma unroll
                for (int j = 0; j < VEC; ++j)
                    if (c + j >= k) x.t[j] = T(0);
            __builtin_nontemporal_store(x.v, reinterpret_cast<u32x4*>(wd_c + dst + i * VEC));
        }
    }
}
}  // namespace

hipError_t launch_export_clipped(const KeepArgs& keep, const void* wg_r, const void* wu_r,
                                 const void* wd_r, void* wg_c, void* wu_c, void* wd_c, int E, int I,
                                 int d, int esize, hipStream_t s) {
    ExportArgs a;
    a.keep = keep;
    int c = 0;
    for (int e = 0; e < kMaxExperts; ++e) {
        a.ch0.v[e] = c;
        if (e < E) c += packed_width(keep.v[e]);
    }
    // enough workgroups per expert to stream its blocks; each loops over the rest
    const dim3 grid(64, E, 3);
    if (esize == 2)
        export_clipped_kernel<bf16_t><<<grid, 256, 0, s>>>(a, (const bf16_t*)wg_r, (const bf16_t*)wu_r,
                                                           (const bf16_t*)wd_r, (bf16_t*)wg_c, (bf16_t*)wu_c,
                                                           (bf16_t*)wd_c, I, d);
    else
        export_clipped_kernel<float><<<grid, 256, 0, s>>>(a, (const float*)wg_r, (const float*)wu_r,
                                                          (const float*)wd_r, (float*)wg_c, (float*)wu_c,
                                                          (float*)wd_c, I, d);
    return hipGetLastError();
}

}  // namespace flexmoe
