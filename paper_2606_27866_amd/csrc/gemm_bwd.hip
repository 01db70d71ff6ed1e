// Backward GEMMs of the channel saliency (FlexMoE Sec. 3.1, Eq. 2) on bf16
// MFMA.  For the loss L = 1/2 sum_t ||Y_t - Y_target_t||^2 and routed expert
// e with dO_a = w_a dY_t (one row per routed assignment):
//   dgrad:  dH[a][c] = sum_n dO_a[n] W_down[n][c]; fused epilogue
//           dG = dH u silu'(g), dU = dH silu(g)           (SwiGLU backward)
//           (the same kernel serves the masked layer's training backward)
//   wgrad:  dW_gate[c][i] = sum_a dG[a][c] x_a[i], dW_up likewise with dU,
//           dW_down[n][c] = sum_a dO_a[n] h_a[c]; fused epilogue
//           s[e][c] += sum over the tile of (theta * dW)^2  (Eq. 2)
// so the weight gradients are never written: each wgrad tile reduces its
// 256 x 256 block of (theta * g)^2 to one partial sum per channel.
//
// All are "NT" GEMMs: A rows and B rows are contiguous in K; the K loop is the
// forward's ping-pong loop over 256 x 256 tiles (mfma_pingpong.h).  In the
// wgrad the MFMA takes the A fragment first, so a lane's accumulator holds one
// B row (a channel) and runs of 4 consecutive A rows, and the weight reads of
// its epilogue are 8-byte accesses.
// On the Qwen1.5-MoE shape with 4096 tokens the loop took, against the one
// before it (both waves of a SIMD on the same step, 32x32x16 MFMAs): wgrad
// 603 -> 600, saliency dgrad 254 -> 228, training dgrad 358 -> 319, dx 338 ->
// 298 us.  With segments on cache lines (below) wgrad takes 517 and the saliency
// dgrad 223.
//   dgrad: A = dO [A][d] (a segment's rows), B = W_down^T [E][I][d] (a
//          transposed copy of the down weights), K = d.
//   wgrad: A = x^T or dO^T [d][ldt], B = dG^T, dU^T or h^T [I][ldt], with a
//          segment's rows as K (columns prow0 .. prow0 + rows of the
//          transposed copies, zero-padded to a multiple of 8; segments start
//          on multiples of TileShape::pad columns).
#include "mfma_pingpong.h"
#include "saliency.h"
#include "train.h"

namespace flexmoe {

namespace {
using namespace mfma;
constexpr int BM = PP_BM, BN = PP_BN, THREADS = PP_THREADS;
constexpr int XCD_GROUP = 8;
static_assert(BM == kSalTile && BN == kSalTile, "host tile counts use kSalTile");

// Requested rows of an operand with rows of `ld` elements: A rows of the tile
// whose first row is row_base (mf: its fragment count), B rows from row_base.
// Rows at or past `valid` (counted from the operand's base) read zeros.
__device__ __forceinline__ void nt_a_rows(int wave, int lane, int row_base, int valid, int ld, int mf,
                                          PPOperands& op) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < PP_ND; ++i) {
            const int r = pp_lds_row(wave, lane, i), row = row_base + pp_a_row(h, r, mf);
            op.col[i] = pp_col(wave, lane, i);
            op.aoff[h][i] = r < 32 * mf && row < valid ? (uint32_t)(((size_t)row * ld + op.col[i]) * 2) : kOOB;
        }
}
__device__ __forceinline__ void nt_b_rows(int wave, int lane, int row_base, int valid, int ld, PPOperands& op) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < PP_ND; ++i) {
            const int row = row_base + h * PP_HALF_ROWS + pp_lds_row(wave, lane, i);
            op.boff[h][i] = row < valid ? (uint32_t)(((size_t)row * ld + pp_col(wave, lane, i)) * 2) : kOOB;
        }
}

// Tile of this workgroup when groups of `group` consecutive tiles go to one
// XCD (workgroup b runs on XCD b % 8): tiles that share operands then share
// that XCD's L2.  The grid is a multiple of 8 * group (xcd_grid).
__device__ __forceinline__ int xcd_tile(int group = XCD_GROUP) {
    const int jb = blockIdx.x >> 3;
    return (jb / group) * (8 * group) + (blockIdx.x & 7) * group + jb % group;
}
long long xcd_grid(long long tiles, int group) { return (tiles + 8LL * group - 1) / (8LL * group) * (8LL * group); }
// Tiles per XCD group of the dgrad kernels: about one routed expert (two
// row tiles x all channel tiles), whose tiles share its rows of dO.
__host__ __device__ __forceinline__ int dgrad_group(int n_ct) { return 2 * n_ct; }

__device__ __forceinline__ float lo_bf16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_bf16(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
}  // namespace

// ---- wgrad + saliency: one tile = 256 hidden units x 256 channels of one
// (matrix, expert) ----------------------------------------------------------
__global__ __launch_bounds__(THREADS, PP_WAVES_PER_SIMD) void sal_wgrad_kernel(SalWgradParams p) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[PP_SMEM];
    // all tiles of one (matrix, expert) on one XCD: they share its x^T (or
    // dO^T) rows and its dG^T (dU^T, h^T) rows
    const int L = xcd_tile(p.nI * p.nM);
    if (L >= 3 * p.E * p.nI * p.nM) return;
    const int mtile = L % p.nM;
    int rest = L / p.nM;
    const int ntile = rest % p.nI;
    rest /= p.nI;
    const int e = rest % p.E, mat = rest / p.E;
    const SegMeta sm = p.seg[p.hs + e];
    const int MP = p.nM * kSalWaveM;  // partial sums per channel
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wm = wave >> 2, wn = wave & 3;
    float* part_out = p.partial + ((size_t)mat * p.E + e) * p.I * MP;

    if (sm.rows == 0) {  // no token reached the expert: its gradient is zero
        if (lane < 32) {
            const int c = ntile * BN + wn * 64 + lane;
            if (c < p.I) part_out[(size_t)c * MP + mtile * kSalWaveM + wm] = 0.f;
            if (c + 32 < p.I) part_out[(size_t)(c + 32) * MP + mtile * kSalWaveM + wm] = 0.f;
        }
        return;
    }

    const bf16_t* A = p.a[mat] + sm.prow0;
    const bf16_t* B = p.b[mat] + sm.prow0;
    const int mf = pp_mf(p.d - mtile * BM);
    PPOperands op;
    op.K = sm.rows;
    op.ra = make_rsrc(A, (size_t)p.d * p.ldt - sm.prow0);
    op.rb[0] = op.rb[1] = make_rsrc(B, (size_t)p.I * p.ldt - sm.prow0);
    nt_a_rows(wave, lane, mtile * BM, p.d, p.ldt, mf, op);
    nt_b_rows(wave, lane, ntile * BN, p.I, p.ldt, op);

    // theta = W[c][m] of the tile's 256 channels x 256 hidden units (gate, up
    // or the transposed down weight), brought into the operand halves by the
    // loop's last eight requests, while its last K tiles are multiplied.
    // Half `half` of slot h holds channels (4h + half) * 32 .. +32, one
    // 512-byte row each; 16-byte chunk pos of row r holds hidden units
    // 8 * (pos ^ r) ..
    const bf16_t* W = p.w[mat] + (size_t)e * p.I * p.d;
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(W, (size_t)p.I * p.d);
    auto theta_tail = [&](int half, int h, unsigned char* dst) {
#pragma unroll
        for (int i = 0; i < PP_ND; ++i) {
            const int tr = wave * 2 * PP_ND + 2 * i + (lane >> 5);  // theta row of the half
            const int c = ntile * BN + (h * 4 + half) * 32 + tr;
            const int m = mtile * BM + ((lane & 31) ^ tr) * 8;
            const uint32_t off = c < p.I && m < p.d ? (uint32_t)(((size_t)c * p.d + m) * 2) : kOOB;
            load_lds16(rw, off, 0, dst + i * PP_RPI * ROWB);
        }
    };
    const int nk = ceil_div(op.K, BK);
    auto theta_half = [&](int half, int h) { return smem + (((nk + h) & 1) * 4 + half) * PP_HALF; };
    pp_by_rows(p.d - mtile * BM, [&](auto tag) {
        constexpr int MF = decltype(tag)::value;
        PPAcc<MF> acc;
        pp_loop<MF, true>(smem, op, wave, lane, acc, theta_tail);
        // the half the loop never refills; its last reads are done
        theta_tail(1, 1, theta_half(1, 1) + wave * (PP_ND * PP_RPI) * ROWB);
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
        barrier_no_fence();  // every wave's theta requests have landed
        // epilogue: lane -> channel, register v -> hidden unit
        // 4(lane/16) + v of a fragment; (theta * dW)^2 summed
        float part[2][2];
#pragma unroll
        for (int bh = 0; bh < 2; ++bh)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                float s = 0.f;
                const int cl = pp_frag_col(bh, wn, j) + (lane & 15);  // channel within the tile
                const unsigned char* trow = theta_half((cl >> 5) & 3, cl >> 7) + (cl & 31) * 512;
#pragma unroll
                for (int ah = 0; ah < 2; ++ah)
#pragma unroll
                    for (int i = 0; i < MF; ++i) {
                        const int ml = pp_frag_row<MF>(ah, wm, i) + (lane >> 4) * 4;
                        const uint2 th = *reinterpret_cast<const uint2*>(
                            trow + (((ml >> 3) ^ (cl & 31)) << 4) + (ml & 7) * 2);
                        const floatx4 g = acc[ah][bh][j * MF + i];
                        const float t0 = lo_bf16(th.x) * g[0];
                        const float t1 = hi_bf16(th.x) * g[1];
                        const float t2 = lo_bf16(th.y) * g[2];
                        const float t3 = hi_bf16(th.y) * g[3];
                        s += (t0 * t0 + t1 * t1) + (t2 * t2 + t3 * t3);
                    }
                s += __shfl_xor(s, 16, 64);
                part[bh][j] = s + __shfl_xor(s, 32, 64);
            }
        if (lane < 16)
#pragma unroll
            for (int bh = 0; bh < 2; ++bh)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int c = ntile * BN + pp_frag_col(bh, wn, j) + lane;
                    if (c < p.I) part_out[(size_t)c * MP + mtile * kSalWaveM + wm] = part[bh][j];
                }
    });
}

// ---- training backward of the masked layer ---------------------------------
namespace {
// Tile L of the training backward's tile list: the shared expert's tiles
// first (ceil(T/256) row tiles x nsh column tiles), then the routed segments'
// (row tiles numbered by SegMeta::rt0, x nr column tiles).  False past the end.
__device__ __forceinline__ bool train_tile(const SegMeta* seg, int hs, int nseg, int T, int Is, int nsh, int nr,
                                           int L, SegMeta& sm, int& mtile, int& ntile, bool with_shared = true) {
    if (hs && with_shared) {
        const int mt = ceil_div(T, BM), sh = mt * nsh;
        if (L < sh) {
            sm = SegMeta{0, T, Is, 0, Is, -1, 0, 0};
            mtile = L % mt;
            ntile = L / mt;
            return true;
        }
        L -= sh;
    }
    int lo = hs, hi = nseg - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (seg[mid].rt0 * nr <= L) lo = mid;
        else hi = mid - 1;
    }
    sm = seg[lo];
    const int mt = ceil_div(sm.rows, BM);
    const int local = L - sm.rt0 * nr;
    if (local >= mt * nr) return false;
    ntile = local / mt;
    mtile = local % mt;
    return true;
}
}  // namespace

// dgrad + SwiGLU backward; tile = 256 rows x 256 channels.  The B fragment
// goes first: lane -> row, registers -> runs of 4 channels.  g and u are read
// in their fragment-blocked layout (a wave's 8-byte reads cover whole
// 128-byte lines); dG and dU are staged through LDS, half of the tile's
// channels at a time, and stored as whole 16-byte pieces.
//   kMode 2 (masked layer's training backward): shared expert included, the
//     mask gradient's partial sums, dG/dU row-major [rows][C] over the kept
//     channels;
//   kMode 1 (channel saliency): routed segments only, every channel kept,
//     dG/dU transposed -- [c][prow0 + r] of [I][ldt], zero in each segment's
//     padding rows -- for the weight-gradient GEMMs.
constexpr int DG_PITCH = BN / 2 + 8;                  // staged row (bf16): 272 bytes, 16-byte aligned
constexpr int DG_STAGE = BM * DG_PITCH * 2;           // one staged array
constexpr int DG_SMEM = (2 * DG_STAGE > PP_SMEM) ? 2 * DG_STAGE : PP_SMEM;
constexpr int DG_TPITCH = BM + 8;                     // transposed staging row (bf16): 4 rows = 16 banks
static_assert(2 * (BN / 2) * DG_TPITCH * 2 <= DG_SMEM, "the transposed staging fits");
static_assert(DG_SMEM <= 160 * 1024, "the dgrad LDS fits one compute unit");

template <int kMode>
__global__ __launch_bounds__(THREADS, PP_WAVES_PER_SIMD) void dgrad_kernel(ActDgradParams p) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[DG_SMEM];
    SegMeta sm;
    int mtile, ntile;
    if (!train_tile(p.seg, p.hs, p.nseg, p.T, p.Is, p.nIs, p.nI, xcd_tile(dgrad_group(p.nI)), sm, mtile, ntile,
                    kMode == 2))
        return;
    const bool shared = sm.e < 0;
    const int C = shared ? p.Is : p.I;  // channels (row length of g, u, dG, dU)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wm = wave >> 2, wn = wave & 3;

    const int row_step = pp_row_step(sm.rows), row0 = mtile * row_step;
    const int tile_rows = min(row_step, sm.rows - row0);
    const int mf = pp_mf(tile_rows);
    PPOperands op;
    op.K = p.d;
    const bf16_t* A = shared ? p.dYs : p.dO + (size_t)sm.row0 * p.d;
    const bf16_t* B = shared ? p.wsdt : p.wdt + (size_t)sm.e * p.I * p.d;
    op.ra = make_rsrc(A, (size_t)sm.rows * p.d);
    op.rb[0] = op.rb[1] = make_rsrc(B, (size_t)C * p.d);
    nt_a_rows(wave, lane, row0, sm.rows, p.d, mf, op);
    nt_b_rows(wave, lane, ntile * BN, C, p.d, op);

    const size_t rbase = shared ? 0 : (size_t)sm.row0;
    const bf16_t* G = shared ? p.Gs : p.G;
    const bf16_t* U = shared ? p.Us : p.U;
    bf16_t* dG = shared ? p.dGs : p.dG;
    bf16_t* dU = shared ? p.dUs : p.dU;
    const int kk = sm.kk;                        // mask: channels below kk are kept
    const int kk8 = min(packed_width(kk), C);    // dG/dU columns the dx GEMM reads
    bf16_t* stg = reinterpret_cast<bf16_t*>(smem);
    bf16_t* stu = stg + (kMode == 2 ? BM * DG_PITCH : (BN / 2) * DG_TPITCH);
    pp_by_rows(tile_rows, [&](auto tag) {
        constexpr int MF = decltype(tag)::value;
        PPAcc<MF> acc;
        pp_loop<MF, false>(smem, op, wave, lane, acc, PPZeroTail{});
        // the operand halves are free once no wave has requests in flight
        barrier_no_fence();
        // epilogue: lane -> row (lane%16 of a fragment), register v ->
        // channel 4(lane/16) + v of a 16-channel fragment
        float msum[2][2][4];
#pragma unroll
        for (int bh = 0; bh < 2; ++bh) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) msum[bh][j][v] = 0.f;
#pragma unroll
            for (int ah = 0; ah < 2; ++ah)
#pragma unroll
            for (int i = 0; i < MF; ++i) {
                const int row = pp_frag_row<MF>(ah, wm, i) + (lane & 15);  // row of the tile
                const int grow = row0 + row;                         // row of the segment
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int cl = pp_frag_col(0, wn, j) + (lane >> 4) * 4;  // staged column of this half
                    const int c0 = ntile * BN + bh * PP_HALF_ROWS + cl;
                    uint32_t dg[2] = {0u, 0u}, du[2] = {0u, 0u};
                    if (grow < sm.rows && c0 < C) {
                        const size_t off = frag_blocked(rbase + grow, c0, C);
                        const uint2 gv = *reinterpret_cast<const uint2*>(G + off);
                        const uint2 uv = *reinterpret_cast<const uint2*>(U + off);
                        const float g[4] = {lo_bf16(gv.x), hi_bf16(gv.x), lo_bf16(gv.y), hi_bf16(gv.y)};
                        const float u[4] = {lo_bf16(uv.x), hi_bf16(uv.x), lo_bf16(uv.y), hi_bf16(uv.y)};
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const float x = g[r];
                            const float sg = 1.0f / (1.0f + __builtin_amdgcn_exp2f(-x * 1.4426950408889634f));
                            const float dh = acc[ah][bh][j * MF + i][r];
                            if constexpr (kMode == 2) msum[bh][j][r] += dh * (x * sg) * u[r];
                            const bool kept = c0 + r < kk;
                            const float vg = kept ? dh * u[r] * (sg * (1.0f + x * (1.0f - sg))) : 0.f;
                            const float vu = kept ? dh * (x * sg) : 0.f;
                            dg[r >> 1] |= (uint32_t)f32_to_bf16(vg) << (16 * (r & 1));
                            du[r >> 1] |= (uint32_t)f32_to_bf16(vu) << (16 * (r & 1));
                        }
                    }
                    if constexpr (kMode == 2) {
                        *reinterpret_cast<uint2*>(stg + row * DG_PITCH + cl) = make_uint2(dg[0], dg[1]);
                        *reinterpret_cast<uint2*>(stu + row * DG_PITCH + cl) = make_uint2(du[0], du[1]);
                    } else {  // staged transposed: [channel][row]
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            stg[(cl + r) * DG_TPITCH + row] = (bf16_t)(dg[r >> 1] >> (16 * (r & 1)));
                            stu[(cl + r) * DG_TPITCH + row] = (bf16_t)(du[r >> 1] >> (16 * (r & 1)));
                        }
                    }
                }
            }
            __syncthreads();
            // staged column cl of half bh is channel ntile*BN + bh*128 + cl
            if constexpr (kMode == 2) {
                for (int k = threadIdx.x; k < BM * (BN / 2 / 8); k += THREADS) {
                    const int row = k / (BN / 2 / 8), cl = (k % (BN / 2 / 8)) * 8;
                    const int grow = row0 + row;
                    const int c = ntile * BN + bh * PP_HALF_ROWS + cl;
                    if (row >= tile_rows || c >= kk8) continue;
                    const size_t o = (rbase + grow) * (size_t)C + c;
                    *reinterpret_cast<u32x4*>(dG + o) = *reinterpret_cast<const u32x4*>(stg + row * DG_PITCH + cl);
                    *reinterpret_cast<u32x4*>(dU + o) = *reinterpret_cast<const u32x4*>(stu + row * DG_PITCH + cl);
                }
            } else {
                // rows up to the segment's padded height (zeros past its rows)
                const int pvalid = packed_width(tile_rows);
                const size_t col = (size_t)sm.prow0 + row0;
                for (int k = threadIdx.x; k < (BN / 2) * (BM / 8); k += THREADS) {
                    const int cl = k / (BM / 8), r0 = (k % (BM / 8)) * 8;
                    const int c = ntile * BN + bh * PP_HALF_ROWS + cl;
                    if (r0 >= pvalid || c >= C) continue;
                    const size_t o = (size_t)c * p.ldt + col + r0;
                    *reinterpret_cast<u32x4*>(dG + o) = *reinterpret_cast<const u32x4*>(stg + cl * DG_TPITCH + r0);
                    *reinterpret_cast<u32x4*>(dU + o) = *reinterpret_cast<const u32x4*>(stu + cl * DG_TPITCH + r0);
                }
            }
            __syncthreads();
        }
        if (kMode == 1 || shared) return;
        // mask-gradient partial sums: over the 16 rows of the lane group
#pragma unroll
        for (int bh = 0; bh < 2; ++bh)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    float t = msum[bh][j][v];
#pragma unroll
                    for (int o = 1; o < 16; o <<= 1) t += __shfl_xor(t, o, 64);
                    msum[bh][j][v] = t;
                }
        if ((lane & 15) == 0) {
            float* out = p.dmp + ((size_t)(sm.rt0 + mtile) * kTrainWaveM + wm) * p.I;
#pragma unroll
            for (int bh = 0; bh < 2; ++bh)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int c = ntile * BN + pp_frag_col(bh, wn, j) + (lane >> 4) * 4 + v;
                        if (c < p.I) out[c] = msum[bh][j][v];
                    }
        }
    });
}

// dX = dG W_gate + dU W_up over the kept channels; tile = 256 rows x 256
// hidden units, one K loop over both products.
__global__ __launch_bounds__(THREADS, PP_WAVES_PER_SIMD) void act_dx_kernel(ActDxParams p) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[PP_SMEM];
    SegMeta sm;
    int mtile, ntile;
    if (!train_tile(p.seg, p.hs, p.nseg, p.T, p.Is, p.nD, p.nD, xcd_tile(dgrad_group(p.nD)), sm, mtile, ntile))
        return;
    const bool shared = sm.e < 0;
    const int C = shared ? p.Is : p.I;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wm = wave >> 2, wn = wave & 3;
    const size_t rbase = shared ? 0 : (size_t)sm.row0;

    const int row_step = pp_row_step(sm.rows), row0 = mtile * row_step;
    const int tile_rows = min(row_step, sm.rows - row0);
    const int mf = pp_mf(tile_rows);
    PPOperands op;
    op.K = sm.kk;
    const bf16_t* Ag = (shared ? p.dGs : p.dG) + rbase * C;
    const bf16_t* Au = (shared ? p.dUs : p.dU) + rbase * C;
    const bf16_t* Bg = shared ? p.wsgt : p.wgt + (size_t)sm.e * p.d * p.I;
    const bf16_t* Bu = shared ? p.wsut : p.wut + (size_t)sm.e * p.d * p.I;
    const PPSecond pairs{Ag, Au, Bg, Bu, (size_t)sm.rows * C, (size_t)p.d * C};
    nt_a_rows(wave, lane, row0, sm.rows, C, mf, op);
    nt_b_rows(wave, lane, ntile * BN, p.d, C, op);
    float* out = (shared ? p.dXs : p.dXr) + rbase * p.d;
    pp_by_rows(tile_rows, [&](auto tag) {
        constexpr int MF = decltype(tag)::value;
        PPAcc<MF> acc;
        pp_loop<MF, false>(smem, op, wave, lane, acc, PPZeroTail{}, pairs);
        // epilogue: lane -> row, registers -> runs of 4 hidden units
#pragma unroll
        for (int ah = 0; ah < 2; ++ah)
#pragma unroll
            for (int i = 0; i < MF; ++i) {
                const int row = row0 + pp_frag_row<MF>(ah, wm, i) + (lane & 15);
                if (row >= sm.rows) continue;
#pragma unroll
                for (int bh = 0; bh < 2; ++bh)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const int n0 = ntile * BN + pp_frag_col(bh, wn, j) + (lane >> 4) * 4;
                        if (n0 >= p.d) continue;
                        *reinterpret_cast<floatx4*>(out + (size_t)row * p.d + n0) = acc[ah][bh][j * MF + i];
                    }
            }
    });
}

hipError_t launch_act_dgrad(const ActDgradParams& p, long long tiles, hipStream_t s) {
    if (tiles <= 0) return hipSuccess;
    const long long g = xcd_grid(tiles, dgrad_group(p.nI));
    dgrad_kernel<2><<<(int)g, THREADS, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_sal_dgrad(const ActDgradParams& p, long long tiles, hipStream_t s) {
    if (tiles <= 0) return hipSuccess;
    const long long g = xcd_grid(tiles, dgrad_group(p.nI));
    dgrad_kernel<1><<<(int)g, THREADS, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_act_dx(const ActDxParams& p, long long tiles, hipStream_t s) {
    if (tiles <= 0) return hipSuccess;
    const long long g = xcd_grid(tiles, dgrad_group(p.nD));
    act_dx_kernel<<<(int)g, THREADS, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_sal_wgrad(const SalWgradParams& p, hipStream_t s) {
    const long long tiles = 3LL * p.E * p.nI * p.nM;
    if (tiles <= 0) return hipSuccess;
    const long long g = xcd_grid(tiles, p.nI * p.nM);
    sal_wgrad_kernel<<<(int)g, THREADS, 0, s>>>(p);
    return hipGetLastError();
}

}  // namespace flexmoe
