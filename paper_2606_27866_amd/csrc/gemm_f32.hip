// fp32 instantiation of the two ragged grouped GEMMs (same segment and tile
// tables as the bf16 path), on the fp32 matrix cores (v_mfma_f32_16x16x4_f32:
// fp32 products and sums; 157 TFLOP/s against 79 for the vector ALUs).
//
// A workgroup of 4 waves owns up to 128 rows x 128 weight rows (64 channels' gate
// and up rows, or 128 output columns) in 80 KB of LDS, two workgroups per
// compute unit.  K tiles of 32 floats are 128-byte LDS rows with XOR-swizzled
// 16-byte chunks (mfma_tile.h), filled by buffer_load ... lds: weights two K
// tiles ahead, token rows one ahead (two in a tile of at most 64 rows); one
// barrier per K tile.  A lane's 16-byte fragment read holds four consecutive
// K of one row and feeds four MFMAs: MFMA q multiplies the K indices
// {4 c + q} of the 16 that the four lane groups hold, the same set on both
// sides.
// MFMA-bound from some tens of rows per expert on: wave w multiplies all rows,
// in steps of 16 (MF = 1..8 fragments), by 32 weight rows, so that the work
// follows the rows more closely than a 2 x 2 arrangement of the waves would
// (steps of 32).
// Against 64 x 64 tiles on the vector ALUs, Qwen1.5-MoE shape with 500 tokens
// and half the channels: 1388 -> 538 us; the 256-wide layer of the parity tests
// with 64 tokens: 98 -> 36 us.
// Operand blocks of 2^29 elements and more (f32_matrix_tiles) keep the
// vector-ALU kernels: the buffer loads address an operand with 32-bit offsets.
#include <type_traits>

#include "mfma_tile.h"

namespace flexmoe {

namespace {
using mfma::kOOB;
constexpr int FBN = kF32MBN2;                  // weight rows per tile
constexpr int FWAVES = 4, FTHREADS = 64 * FWAVES;
constexpr int FBK = mfma::ROWB / 4;            // K elements per LDS row
constexpr int FRPI = 64 / mfma::CHUNKS;        // LDS rows one DMA instruction fills
constexpr int FNB = FBN / (FWAVES * FRPI);     // weight DMA instructions per wave and K tile
constexpr int FB_STAGE = FBN * mfma::ROWB;     // 16 KB
constexpr int FB_STAGES = 3;
constexpr int FA_BYTES = 2 * kF32MBM * mfma::ROWB;  // two stages of 128 token rows or three of 64
constexpr int F32_SMEM = FB_STAGES * FB_STAGE + FA_BYTES;
static_assert(2 * F32_SMEM <= 160 * 1024, "two workgroups share a compute unit's LDS");
static_assert(2 * kF32MBN1 == FBN && kF32MBM == 128, "the tile tables are built with these widths");

__device__ __forceinline__ __amdgpu_buffer_rsrc_t f32_rsrc(const float* base, size_t elems) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), (short)0, (int)(elems * 4), 0x00020000);
}
}  // namespace

template <bool kGateUp>
__device__ __forceinline__ void f32_tile(const Gemm1Params<float>& p1, const Gemm2Params<float>& p2,
                                         unsigned char* smem) {
    using namespace mfma;
    const int d = kGateUp ? p1.d : p2.d;
    int s, local;
    SegMeta sm;
    if (!(kGateUp ? tile_of(p1, blockIdx.x, s, sm, local) : tile_of(p2, blockIdx.x, s, sm, local))) return;
    const bool shared = sm.e < 0;
    const int bm = kGateUp ? p1.bm : p2.bm;  // 32, 64 or 128
    const int mt = ceil_div(sm.rows, bm);
    const int mtile = local % mt, ntile = local / mt;
    const int row0 = mtile * bm, tile_rows = min(bm, sm.rows - row0);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;

    int K, lda, ldw;
    __amdgpu_buffer_rsrc_t ra, rb;
    if constexpr (kGateUp) {
        K = lda = ldw = d;
        const RoutedWeights rw = shared ? RoutedWeights{0, p1.Is, 0} : routed_weights(p1, sm);
        // waves 0 and 1 request the gate rows, waves 2 and 3 the up rows
        const float* W = (wave < FWAVES / 2 ? (shared ? p1.sg : p1.wg) : (shared ? p1.su : p1.wu)) + rw.base;
        ra = f32_rsrc(p1.x, (size_t)p1.tokens * d);
        rb = f32_rsrc(W, (size_t)rw.rows * d);
    } else {
        K = sm.kg;
        const RoutedWeights rw = shared ? RoutedWeights{0, 0, p2.Is} : routed_weights(p2, sm);
        lda = shared ? p2.Is : p2.I;
        ldw = rw.ldd;
        ra = f32_rsrc(shared ? p2.Hs : p2.H + (size_t)sm.row0 * p2.I, (size_t)(shared ? p2.tokens : sm.rows) * lda);
        rb = f32_rsrc(shared ? p2.sd : p2.wd + rw.base, (size_t)d * ldw);
    }
    // DMA instruction i of a wave fills 8 LDS rows; lane -> row lane/8, LDS
    // chunk lane%8, which holds the row's K chunk swz(row, lane%8) (row bits
    // 1..3: it depends on the parity of i alone).  Masked rows read zeros.
    uint32_t boff[FNB];
    int col[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) col[i] = swz(i * FRPI + lane / CHUNKS, lane % CHUNKS) * 4;
#pragma unroll
    for (int i = 0; i < FNB; ++i) {
        const int r = wave * (FNB * FRPI) + i * FRPI + lane / CHUNKS;
        const int n = kGateUp ? ntile * kF32MBN1 + (r & (kF32MBN1 - 1)) : ntile * FBN + r;
        boff[i] = n < (kGateUp ? sm.kg : d) ? (uint32_t)(((size_t)n * ldw + col[i & 1]) * 4) : kOOB;
    }
    const int nk = ceil_div(K, FBK);
    const int lr = lane & 15, lc = lane >> 4;

    // The K loop and epilogue for a tile of MF 16-row fragments.
    auto run = [&](auto mf_tag) {
        constexpr int MF = decltype(mf_tag)::value;
        constexpr int AROWS = MF > 4 ? 128 : 64;     // staged token rows
        constexpr int DA = MF > 4 ? 1 : 2;           // K tiles the token rows are requested ahead
        constexpr int NA = AROWS / (FWAVES * FRPI);  // token-row DMA instructions per wave and K tile
        constexpr int A_STAGE = AROWS * ROWB;
        static_assert((DA + 1) * A_STAGE <= FA_BYTES, "the token-row stages fit");
        unsigned char* sA = smem + FB_STAGES * FB_STAGE;
        uint32_t aoff[NA];
        int src[NA];
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            src[i] = row0 + wave * (NA * FRPI) + i * FRPI + lane / CHUNKS;
            // rows past the segment read its last row's entry, unused
            if (kGateUp && !shared) src[i] = p1.perm[sm.row0 + min(src[i], sm.rows - 1)];
        }
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int r = wave * (NA * FRPI) + i * FRPI + lane / CHUNKS;
            if (kGateUp && !shared) src[i] = (int)min((unsigned)(src[i] / p1.top_k), (unsigned)(p1.tokens - 1));
            aoff[i] = r < tile_rows ? (uint32_t)(((size_t)src[i] * lda + col[i & 1]) * 4) : kOOB;
        }
        // past the end every lane's offset is kOOB: the count of outstanding
        // requests stays exact
        auto request_a = [&](int kt, int stage) {
            const int lim = K - kt * FBK;
#pragma unroll
            for (int i = 0; i < NA; ++i)
                load_lds16(ra, col[i & 1] < lim ? aoff[i] : kOOB, (uint32_t)(kt * FBK) * 4u,
                           sA + stage * A_STAGE + (wave * NA + i) * (FRPI * ROWB));
        };
        auto request_b = [&](int kt, int stage) {
            const int lim = K - kt * FBK;
#pragma unroll
            for (int i = 0; i < FNB; ++i)
                load_lds16(rb, col[i & 1] < lim ? boff[i] : kOOB, (uint32_t)(kt * FBK) * 4u,
                           smem + stage * FB_STAGE + (wave * FNB + i) * (FRPI * ROWB));
        };
        floatx4 acc[2][MF];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < MF; ++i) acc[j][i] = floatx4{0.f, 0.f, 0.f, 0.f};
        // weight row of fragment j: gate rows, then the same channels' up
        // rows, or 32 output columns
        auto brow = [&](int j) { return kGateUp ? j * kF32MBN1 + wave * 16 : wave * 32 + j * 16; };
        request_a(0, 0);
        request_b(0, 0);
        if constexpr (DA == 2) request_a(1, 1);
        request_b(1, 1);
        int sa = 0, sb = 0;  // stages of tile kt
        for (int kt = 0; kt < nk; ++kt) {
            // tile kt is in when only the requests of tile kt + 1 are
            // outstanding; this wave's LDS reads of tile kt - 1 are done, so
            // after the barrier its stages may be refilled
            __builtin_amdgcn_s_waitcnt(waitcnt_vm(DA == 2 ? NA + FNB : FNB) & kWaitLgkm0);
            barrier_no_fence();
            request_a(kt + DA, sa == 0 ? DA : sa - 1);
            request_b(kt + 2, sb == 0 ? FB_STAGES - 1 : sb - 1);
            const unsigned char* a = sA + sa * A_STAGE;
            const unsigned char* b = smem + sb * FB_STAGE;
            floatx4 fa[2][MF], fb[2][2];
#pragma unroll
            for (int st = 0; st < 2; ++st) {
#pragma unroll
                for (int j = 0; j < 2; ++j) fb[st][j] = __builtin_bit_cast(floatx4, lds_frag(b, brow(j) + lr, st * 4 + lc));
#pragma unroll
                for (int i = 0; i < MF; ++i) fa[st][i] = __builtin_bit_cast(floatx4, lds_frag(a, i * 16 + lr, st * 4 + lc));
            }
            if (!kGateUp && (K & 3) && kt == nk - 1) {
                // a reduction that ends inside a chunk: the weights past it
                // are real values, and a product with one that is not finite
                // would not be zero
#pragma unroll
                for (int st = 0; st < 2; ++st)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (kt * FBK + (st * 4 + lc) * 4 + q >= K) {
#pragma unroll
                            for (int j = 0; j < 2; ++j) fb[st][j][q] = 0.f;
                        }
            }
#pragma unroll
            for (int st = 0; st < 2; ++st)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
#pragma unroll
                        for (int i = 0; i < MF; ++i)
                            acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[st][j][q], fa[st][i][q], acc[j][i], 0, 0, 0);
            sa = sa == DA ? 0 : sa + 1;
            sb = sb == FB_STAGES - 1 ? 0 : sb + 1;
        }
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));  // no DMA may outlive the workgroup's LDS

        // lane -> row lane%16 of a fragment, registers -> 4 consecutive weight
        // rows from 4*(lane/16): 16-byte stores
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            const int row = row0 + i * 16 + lr;
            if (row >= sm.rows) continue;
            if constexpr (kGateUp) {
                const int ldh = shared ? p1.Is : p1.I;
                float* hr = (shared ? p1.Hs : p1.H + (size_t)sm.row0 * p1.I) + (size_t)row * ldh;
                // channels from kk to the GEMM width rounded up to 8 are
                // written as zeros (the down GEMM reads whole 16-byte chunks)
                const int kk8 = min((sm.kg + 7) & ~7, ldh);
                const int ch = ntile * kF32MBN1 + wave * 16 + lc * 4;
                if (ch >= kk8) continue;
                floatx4 h;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float g = acc[0][i][v];
                    h[v] = ch + v < sm.kk ? g / (1.0f + expf(-g)) * acc[1][i][v] : 0.f;
                }
                *reinterpret_cast<floatx4*>(hr + ch) = h;
            } else {
                float* orow = (shared ? p2.Os : p2.O + (size_t)sm.row0 * d) + (size_t)row * d;
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int n = ntile * FBN + brow(j) + lc * 4;
                    if (n < d) *reinterpret_cast<floatx4*>(orow + n) = acc[j][i];
                }
            }
        }
    };
    switch (ceil_div(tile_rows, 16)) {
        case 1: run(std::integral_constant<int, 1>{}); break;
        case 2: run(std::integral_constant<int, 2>{}); break;
        case 3: run(std::integral_constant<int, 3>{}); break;
        case 4: run(std::integral_constant<int, 4>{}); break;
        case 5: run(std::integral_constant<int, 5>{}); break;
        case 6: run(std::integral_constant<int, 6>{}); break;
        case 7: run(std::integral_constant<int, 7>{}); break;
        default: run(std::integral_constant<int, 8>{}); break;
    }
}

__global__ __launch_bounds__(FTHREADS, 2) void gemm1_f32_kernel(Gemm1Params<float> p) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[F32_SMEM];
    f32_tile<true>(p, Gemm2Params<float>{}, smem);
}
__global__ __launch_bounds__(FTHREADS, 2) void gemm2_f32_kernel(Gemm2Params<float> p) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[F32_SMEM];
    f32_tile<false>(Gemm1Params<float>{}, p, smem);
}

// ---- vector-ALU tiles (64 x 64, 4 x 4 outputs per thread) for operand blocks
// past the buffer loads' reach
namespace {
constexpr int BM = kF32BM, BN = kF32BN, BK = 16;
}

__global__ __launch_bounds__(256) void gemm1_f32_valu_kernel(Gemm1Params<float> p) {
    __shared__ float As[BK][BM + 4];
    __shared__ float Bg[BK][BN + 4];
    __shared__ float Bu[BK][BN + 4];
    int s, local;
    SegMeta sm;
    if (!tile_of(p, blockIdx.x, s, sm, local)) return;
    const int mt = ceil_div(sm.rows, BM);
    const int mtile = local % mt, ntile = local / mt;
    const bool shared = sm.e < 0;
    const size_t wofs = shared ? 0 : routed_weights(p, sm).base;
    const float* Wg = (shared ? p.sg : p.wg) + wofs;
    const float* Wu = (shared ? p.su : p.wu) + wofs;

    const int tid = threadIdx.x;
    const int lr = tid >> 2, lk = (tid & 3) * 4;
    const int row = mtile * BM + lr;
    const float* asrc = nullptr;
    if (row < sm.rows) {
        const int t = shared ? row : (int)min((unsigned)(p.perm[sm.row0 + row] / p.top_k), (unsigned)(p.tokens - 1));
        asrc = p.x + (size_t)t * p.d;
    }
    const int ch = ntile * BN + lr;
    const float* gsrc = ch < sm.kg ? Wg + (size_t)ch * p.d : nullptr;  // channels the GEMM computes
    const float* usrc = ch < sm.kg ? Wu + (size_t)ch * p.d : nullptr;

    const int ty = tid >> 4, tx = tid & 15;
    float ag[4][4] = {}, au[4][4] = {};
    const float4 z4 = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k0 = 0; k0 < p.d; k0 += BK) {
        const bool kin = k0 + lk < p.d;
        const float4 a = (asrc && kin) ? *reinterpret_cast<const float4*>(asrc + k0 + lk) : z4;
        const float4 g = (gsrc && kin) ? *reinterpret_cast<const float4*>(gsrc + k0 + lk) : z4;
        const float4 u = (usrc && kin) ? *reinterpret_cast<const float4*>(usrc + k0 + lk) : z4;
        As[lk + 0][lr] = a.x; As[lk + 1][lr] = a.y; As[lk + 2][lr] = a.z; As[lk + 3][lr] = a.w;
        Bg[lk + 0][lr] = g.x; Bg[lk + 1][lr] = g.y; Bg[lk + 2][lr] = g.z; Bg[lk + 3][lr] = g.w;
        Bu[lk + 0][lr] = u.x; Bu[lk + 1][lr] = u.y; Bu[lk + 2][lr] = u.z; Bu[lk + 3][lr] = u.w;
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < BK; ++kk) {
            float av[4], gv[4], uv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) av[i] = As[kk][ty * 4 + i];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                gv[j] = Bg[kk][tx * 4 + j];
                uv[j] = Bu[kk][tx * 4 + j];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    ag[i][j] = fmaf(av[i], gv[j], ag[i][j]);
                    au[i][j] = fmaf(av[i], uv[j], au[i][j]);
                }
        }
        __syncthreads();
    }
    float* Hb = shared ? p.Hs : p.H + (size_t)sm.row0 * p.I;
    const int ldh = shared ? p.Is : p.I;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = mtile * BM + ty * 4 + i;
            const int c = ntile * BN + tx * 4 + j;
            if (r < sm.rows && c < sm.kg) {  // channels [kk, kg) are written as zeros
                const float g = ag[i][j];
                Hb[(size_t)r * ldh + c] = c < sm.kk ? g / (1.0f + expf(-g)) * au[i][j] : 0.0f;
            }
        }
}

__global__ __launch_bounds__(256) void gemm2_f32_valu_kernel(Gemm2Params<float> p) {
    __shared__ float As[BK][BM + 4];
    __shared__ float Bs[BK][BN + 4];
    int s, local;
    SegMeta sm;
    if (!tile_of(p, blockIdx.x, s, sm, local)) return;
    const int mt = ceil_div(sm.rows, BM);
    const int mtile = local % mt, ntile = local / mt;
    const bool shared = sm.e < 0;
    const float* Hb = shared ? p.Hs : p.H + (size_t)sm.row0 * p.I;
    const RoutedWeights rw = shared ? RoutedWeights{0, 0, p.Is} : routed_weights(p, sm);
    const int ldh = shared ? p.Is : p.I;  // H row stride
    const float* Wd = shared ? p.sd : p.wd + rw.base;
    const int K = sm.kg;

    const int tid = threadIdx.x;
    const int lr = tid >> 2, lk = (tid & 3) * 4;
    const int row = mtile * BM + lr;
    const float* asrc = row < sm.rows ? Hb + (size_t)row * ldh : nullptr;
    const int n = ntile * BN + lr;
    const float* bsrc = n < p.d ? Wd + (size_t)n * rw.ldd : nullptr;

    const int ty = tid >> 4, tx = tid & 15;
    float acc[4][4] = {};
    for (int k0 = 0; k0 < K; k0 += BK) {
        const int kb = k0 + lk;
        float a[4] = {0.f, 0.f, 0.f, 0.f}, b[4] = {0.f, 0.f, 0.f, 0.f};
        if (kb < K) {  // kb % 4 == 0 and the strides are multiples of 8: the vector is in bounds
            const float4 va = asrc ? *reinterpret_cast<const float4*>(asrc + kb) : make_float4(0.f, 0.f, 0.f, 0.f);
            const float4 vb = bsrc ? *reinterpret_cast<const float4*>(bsrc + kb) : make_float4(0.f, 0.f, 0.f, 0.f);
            a[0] = va.x; a[1] = va.y; a[2] = va.z; a[3] = va.w;
            b[0] = vb.x; b[1] = vb.y; b[2] = vb.z; b[3] = vb.w;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (kb + q >= K) a[q] = b[q] = 0.f;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            As[lk + q][lr] = a[q];
            Bs[lk + q][lr] = b[q];
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < BK; ++kk) {
            float av[4], bv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) av[i] = As[kk][ty * 4 + i];
#pragma unroll
            for (int j = 0; j < 4; ++j) bv[j] = Bs[kk][tx * 4 + j];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(av[i], bv[j], acc[i][j]);
        }
        __syncthreads();
    }
    float* Ob = shared ? p.Os : p.O + (size_t)sm.row0 * p.d;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = mtile * BM + ty * 4 + i;
            const int c = ntile * BN + tx * 4 + j;
            if (r < sm.rows && c < p.d) Ob[(size_t)r * p.d + c] = acc[i][j];
        }
}

hipError_t launch_gemm1_f32(const Gemm1Params<float>& p, int grid, hipStream_t s, bool matrix) {
    if (grid <= 0) return hipSuccess;
    if (matrix) gemm1_f32_kernel<<<grid, FTHREADS, 0, s>>>(p);
    else gemm1_f32_valu_kernel<<<grid, 256, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_gemm2_f32(const Gemm2Params<float>& p, int grid, hipStream_t s, bool matrix) {
    if (grid <= 0) return hipSuccess;
    if (matrix) gemm2_f32_kernel<<<grid, FTHREADS, 0, s>>>(p);
    else gemm2_f32_valu_kernel<<<grid, 256, 0, s>>>(p);
    return hipGetLastError();
}

}  // namespace flexmoe
