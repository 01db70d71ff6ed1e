// Large-tile ragged grouped GEMMs on bf16 MFMA for prefill-sized token counts.
//
// The gate/up GEMM with fused SwiGLU and the down GEMM with the reduction
// truncated to k_e (FlexMoE Eq. 4), shaped for gfx950:
//   - 256 x 256 workgroup tile (rows x weight rows), K tile 64, 8 waves, two
//     per SIMD, that alternate between the matrix core and the memory work of
//     their next fragments: the ping-pong K loop of mfma_pingpong.h (128 KB
//     of LDS, 16x16x32 MFMAs).  Against the loop before it (both waves of a
//     SIMD doing the same step, 32x32x16 MFMAs, 160 KB of LDS) the
//     Mixtral-shaped layer at 16384 tokens and half the channels went from
//     4.83 to 4.32 ms, the Qwen2-57B-shaped one at 8192 tokens and 60 %
//     from 5.14 to 4.62 ms.
//   - operands go from global memory straight into LDS (buffer_load ... lds,
//     16 bytes per lane): no VGPRs stage them and no ds_write is issued.
//     Each lane's offset into the operand is fixed for the whole reduction;
//     the K position is a scalar offset.  Rows outside a segment, channels at
//     or past k_e and K chunks past the end use an offset outside the buffer
//     descriptor, for which the hardware returns zeros.
//   - each 128-byte LDS row (64 bf16 of K) stores its eight 16-byte chunks
//     XOR-swizzled by bits 1..3 of the row index, so the 16 lanes served in
//     one LDS cycle of a fragment read hit 64 distinct banks.
//   - tiles are numbered segment-major (shared expert first: its reductions
//     are the longest), inside a segment in groups of four row tiles (all
//     columns of a group, a column's row tiles consecutive); runs of 8
//     consecutive tiles (32 for a gate/up launch with no concurrent launch
//     beside it) go to one XCD (workgroup b runs on XCD b % 8), interleaving
//     the XCDs run by run, so that the tiles an XCD runs at once share
//     token-row and weight panels in its L2 while the work stays balanced.
// gate/up: a workgroup tile is 256 rows x 128 channels; B half 0 holds the 128
//   gate rows and B half 1 the 128 up rows of those channels, so the gate and
//   up accumulators of a channel sit in the same lane.
// down: a workgroup tile is 256 rows x 256 output columns.  When the shared
//   expert alone has too few tiles to fill the chip, its reduction over I_s
//   is split into chunks whose partial rows the combine adds in chunk order.
// A segment's last row tile often holds far fewer than 256 rows (a routed
// expert gets a few hundred tokens).  A tile with R rows runs the variant in
// which each wave multiplies ceil(R/64) fragments of 16 rows per A half, so
// MFMA work follows the rows at a 64-row granularity; the loads stay the same
// (rows past the segment read zeros).
#include "mfma_pingpong.h"

namespace flexmoe {

namespace {
using namespace mfma;
constexpr int BM = PP_BM, BN = PP_BN, THREADS = PP_THREADS;
constexpr int NSB = 2;                      // K tiles staged in LDS
static_assert(PP_SMEM == NSB * (BM + BN) * ROWB, "the K loop stages NSB tiles of both operands");
constexpr int XCD_GROUP = 8;                // consecutive tiles kept on one XCD (default)
constexpr int ROW_GROUP = 4;                // row tiles of a segment walked before the next column
}  // namespace

// Saliency forward: the tile's h (256 rows x 128 channels) written
// transposed through an LDS staging tile.
constexpr int TROW = 256 + 8;  // staging row pitch (bf16): 4 rows apart = 16 banks apart
static_assert(128 * TROW * 2 <= PP_SMEM, "the staging tile fits in the operand stages");

template <int MF>
__device__ __forceinline__ void train_store_h_transposed(const Gemm1Params<bf16_t>& p, const SegMeta& sm,
                                                         const PPAcc<MF>& acc, unsigned char* smem, int row0,
                                                         int tile_rows, int ntile, int wave, int lane) {
    const int wm = wave >> 2, wn = wave & 3;
    bf16_t* st = reinterpret_cast<bf16_t*>(smem);
    const int pvalid = packed_width(tile_rows);  // rows written: the segment's last tile pads it to 8
    const int ch_tile = ntile * (BN / 2);
    // the operand stages are free once no wave has requests in flight
    barrier_no_fence();
#pragma unroll
    for (int ah = 0; ah < 2; ++ah)
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            const int row = pp_frag_row<MF>(ah, wm, i) + (lane & 15);
            const bool real = row < tile_rows;
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int cl = pp_frag_col(0, wn, j) + (lane >> 4) * 4 + r;
                    const float g = acc[ah][0][j * MF + i][r], u = acc[ah][1][j * MF + i][r];
                    st[cl * TROW + row] = real ? f32_to_bf16(silu_fast(g) * u) : (bf16_t)0;
                }
        }
    __syncthreads();
    bf16_t* out = p.ht + (size_t)sm.prow0 + row0;
    for (int k = threadIdx.x; k < (BN / 2) * (BM / 8); k += THREADS) {
        const int cl = k / (BM / 8), r0 = (k % (BM / 8)) * 8;
        const int ch = ch_tile + cl;
        if (r0 >= pvalid || ch >= sm.kg) continue;
        *reinterpret_cast<u32x4*>(out + (size_t)ch * p.ldt + r0) =
            *reinterpret_cast<const u32x4*>(st + cl * TROW + r0);
    }
}

// kTrain: 0 = inference; 1 = also g and u of the routed rows
// (fragment-blocked) and their h transposed (channel saliency); 2 = also g
// and u of every row, fragment-blocked (the masked layer's training backward).
// XG: consecutive tiles kept on one XCD (XCD_GROUP, or 32 for a gate/up
// launch with the GPU to itself, see gemm1_big_kernel).
template <bool kGateUp, int kTrain = 0, int XG = XCD_GROUP>
__device__ __forceinline__ void big_tile(const Gemm1Params<bf16_t>& p1, const Gemm2Params<bf16_t>& p2,
                                         unsigned char* smem) {
    const int d = kGateUp ? p1.d : p2.d;

    // tile numbering: XCD x = b % 8 takes runs of XG consecutive tiles
    const int jb = blockIdx.x >> 3;
    const int L = (jb / XG) * (8 * XG) + (blockIdx.x & 7) * XG + jb % XG;
    int s, local;
    SegMeta sm;
    if (!(kGateUp ? tile_of(p1, L, s, sm, local) : tile_of(p2, L, s, sm, local))) return;
    // A segment's tiles form an mt x nt grid (row tiles x channel or output
    // column tiles); the down GEMM of a split shared expert has one grid per
    // reduction chunk, chunk `split` after chunk split-1.  Inside a grid the
    // tiles go in groups of ROW_GROUP row tiles: all columns of a group, each
    // column's row tiles consecutive, then the next group.  An XCD's 32
    // concurrent tiles (four runs of 8 from consecutive rounds over the 8
    // XCDs, or one run of 32) then share about ROW_GROUP token-row panels
    // and 8 weight panels through its L2, instead of needing up to 32
    // token-row panels and 4 weight panels: the L2 misses of the
    // Mixtral-shaped gate/up launch drop from 13.3 GB (one row tile after
    // another) to 9.5 GB with runs of 8 and 6.8 GB with runs of 32.
    const int mt = ceil_div(sm.rows, BM);
    const int nt = kGateUp ? ceil_div(sm.kg, BN / 2) : ceil_div(d, BN);
    const int split = kGateUp ? 0 : local / (mt * nt);
    const int loc = kGateUp ? local : local - split * mt * nt;
    const int grp = loc / (ROW_GROUP * nt);
    const int rem = loc - grp * ROW_GROUP * nt;
    const int grows = min(ROW_GROUP, mt - grp * ROW_GROUP);  // row tiles of this group
    const int ntile = rem / grows, mtile = grp * ROW_GROUP + rem % grows;
    const bool shared = sm.e < 0;

    // the wave index is uniform: keeping it in a scalar register makes every
    // LDS destination address (M0) scalar arithmetic
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;

    // ---- buffer descriptors and the rows this lane requests (PPOperands).
    // Masked rows (outside the segment, channels at or past k_e, columns past
    // d) get an offset past the descriptor's extent, for which the load
    // returns zeros.
    const int row_step = pp_row_step(sm.rows), row0 = mtile * row_step;
    const int tile_rows = min(row_step, sm.rows - row0);
    const int mf = pp_mf(tile_rows);
    PPOperands op;
#pragma unroll
    for (int i = 0; i < PP_ND; ++i) op.col[i] = pp_col(wave, lane, i);
    // tile row of each A row this lane requests; rows past the tile are masked
    int arow[2][PP_ND];
    bool aval[2][PP_ND];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < PP_ND; ++i) {
            const int r = pp_lds_row(wave, lane, i);
            arow[h][i] = pp_a_row(h, r, mf);
            aval[h][i] = r < 32 * mf && arow[h][i] < tile_rows;
        }
    if constexpr (kGateUp) {
        op.K = d;
        const RoutedWeights rw = shared ? RoutedWeights{0, p1.Is, 0} : routed_weights(p1, sm);
        op.ra = make_rsrc(p1.x, (size_t)p1.tokens * d);
        op.rb[0] = make_rsrc((shared ? p1.sg : p1.wg) + rw.base, (size_t)rw.rows * d);
        op.rb[1] = make_rsrc((shared ? p1.su : p1.wu) + rw.base, (size_t)rw.rows * d);
        // token of each A row: every lane loads its rows' entries of the
        // permutation (rows past the segment read its last row's, unused), so
        // the loads are in flight together rather than one after another
        int tok[2][PP_ND];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < PP_ND; ++i) {
                tok[h][i] = row0 + arow[h][i];
                if (!shared) tok[h][i] = p1.perm[sm.row0 + min(tok[h][i], sm.rows - 1)];
            }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < PP_ND; ++i) {
                const int c = op.col[i];
                const int t = shared ? tok[h][i]
                                     : (int)min((unsigned)(tok[h][i] / p1.top_k), (unsigned)(p1.tokens - 1));
                op.aoff[h][i] = aval[h][i] ? (uint32_t)(((size_t)t * d + c) * 2) : kOOB;
                const int ch = ntile * (BN / 2) + pp_lds_row(wave, lane, i);
                op.boff[h][i] = ch < sm.kg ? (uint32_t)(((size_t)ch * d + c) * 2) : kOOB;
            }
    } else {
        const int kbeg = shared && p2.ks2 > 0 ? split * p2.ks2 : 0;
        op.K = shared && p2.ks2 > 0 ? min(sm.kg - kbeg, p2.ks2) : p2.kept_only ? sm.kk : sm.kg;
        const RoutedWeights rw = shared ? RoutedWeights{0, 0, p2.Is} : routed_weights(p2, sm);
        const int ldh = shared ? p2.Is : p2.I;  // H row stride
        const int ldw = rw.ldd;                 // W_down row stride
        const int hrows = shared ? p2.tokens : sm.rows;
        const bf16_t* Hb = (shared ? p2.Hs : p2.H + (size_t)sm.row0 * p2.I) + kbeg;
        const bf16_t* Wd = (shared ? p2.sd : p2.wd + rw.base) + kbeg;
        op.ra = make_rsrc(Hb, (size_t)hrows * ldh - kbeg);
        op.rb[0] = op.rb[1] = make_rsrc(Wd, (size_t)d * ldw - kbeg);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < PP_ND; ++i) {
                const int c = op.col[i];
                const int row = row0 + arow[h][i];
                op.aoff[h][i] = aval[h][i] ? (uint32_t)(((size_t)row * ldh + c) * 2) : kOOB;
                const int n = ntile * BN + h * PP_HALF_ROWS + pp_lds_row(wave, lane, i);
                op.boff[h][i] = n < d ? (uint32_t)(((size_t)n * ldw + c) * 2) : kOOB;
            }
    }

    const int wm = wave >> 2, wn = wave & 3;

    // The K loop and epilogue for tiles whose waves multiply MF 16-row
    // fragments of each A half.
    auto run = [&](auto mf_tag) {
        constexpr int MF = decltype(mf_tag)::value;
        PPAcc<MF> acc;
        pp_loop<MF, false>(smem, op, wave, lane, acc, PPZeroTail{});

        // ---- epilogue: lane -> row lane%16 of a fragment, registers -> 4
        // consecutive channels (or output columns) from 4*(lane/16), stored as
        // one 8-byte write.
        const int sub = (lane >> 4) * 4;
        if constexpr (kGateUp) {
            bf16_t* Hb = shared ? p1.Hs : p1.H + (size_t)sm.row0 * p1.I;
            const int ldh = shared ? p1.Is : p1.I;
            // channels [kk, kk8) are written as zeros, kk8 = the GEMM width
            // rounded up to 8 (the down GEMM reads whole 16-byte chunks); kk8
            // and the runs are multiples of 8 and 4, so a run is wholly inside
            // or outside
            const int kk8 = min((sm.kg + 7) & ~7, ldh);
            // g and u for the training backward, in the fragment-blocked
            // layout (common.h) over the routed row space (or the tokens)
            const bool keep_gu = kTrain == 2 || (kTrain == 1 && !shared);
            bf16_t* Gb = shared ? p1.Gs : p1.G;
            bf16_t* Ub = shared ? p1.Us : p1.U;
            const size_t rbase = shared ? 0 : (size_t)sm.row0;
#pragma unroll
            for (int ah = 0; ah < 2; ++ah)
#pragma unroll
                for (int i = 0; i < MF; ++i) {
                    const int row = row0 + pp_frag_row<MF>(ah, wm, i) + (lane & 15);
                    if (row >= sm.rows) continue;
                    bf16_t* hr = Hb + (size_t)row * ldh;
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const int ch = ntile * (BN / 2) + pp_frag_col(0, wn, j) + sub;
                        if (ch >= kk8) continue;
                        const floatx4 g = acc[ah][0][j * MF + i], u = acc[ah][1][j * MF + i];
                        float h[4];
#pragma unroll
                        for (int v = 0; v < 4; ++v) h[v] = ch + v < sm.kk ? silu_fast(g[v]) * u[v] : 0.f;
                        *reinterpret_cast<uint2*>(hr + ch) = make_uint2(pack_bf16x2(h[0], h[1]), pack_bf16x2(h[2], h[3]));
                        if (keep_gu && ch < sm.kg) {
                            const size_t off = frag_blocked(rbase + row, ch, ldh);
                            *reinterpret_cast<uint2*>(Gb + off) = make_uint2(pack_bf16x2(g[0], g[1]), pack_bf16x2(g[2], g[3]));
                            *reinterpret_cast<uint2*>(Ub + off) = make_uint2(pack_bf16x2(u[0], u[1]), pack_bf16x2(u[2], u[3]));
                        }
                    }
                }
            if constexpr (kTrain == 1) {
                // h transposed for the weight-gradient GEMMs, element
                // [c][prow0 + row], zero in the rows up to the segment's padded
                // height, staged through LDS as a [128 channels][256 rows] tile
                // so that global stores are whole 16-byte row pieces
                if (!shared) train_store_h_transposed<MF>(p1, sm, acc, smem, row0, tile_rows, ntile, wave, lane);
            }
        } else {
            bf16_t* Ob = shared ? p2.Os + (size_t)split * p2.tokens * d : p2.O + (size_t)sm.row0 * d;
#pragma unroll
            for (int ah = 0; ah < 2; ++ah)
#pragma unroll
                for (int i = 0; i < MF; ++i) {
                    const int row = row0 + pp_frag_row<MF>(ah, wm, i) + (lane & 15);
                    if (row >= sm.rows) continue;
                    bf16_t* orow = Ob + (size_t)row * d;
#pragma unroll
                    for (int bh = 0; bh < 2; ++bh)
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            const int n = ntile * BN + pp_frag_col(bh, wn, j) + sub;
                            if (n >= d) continue;
                            const floatx4 o = acc[ah][bh][j * MF + i];
                            *reinterpret_cast<uint2*>(orow + n) = make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
                        }
                }
        }
    };

    pp_by_rows(tile_rows, run);
}

// XG = 32 when no side-stream launch runs at all: the L2 misses drop by 29 %
// and the layer step by about 1 % (Mixtral and Qwen2-57B shapes); beside a
// side-stream launch the longer runs were 0.5 % slower.  The down GEMM keeps
// runs of 8: its segments' reductions differ, and longer runs left the XCDs
// unevenly loaded at the end.
template <int XG>
__global__ __launch_bounds__(THREADS, PP_WAVES_PER_SIMD) void gemm1_big_kernel(Gemm1Params<bf16_t> p) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[PP_SMEM];
    big_tile<true, 0, XG>(p, Gemm2Params<bf16_t>{}, smem);
}

// The gate/up GEMM of the channel saliency: the same tiles, plus g and u of
// the routed rows (fragment-blocked) and their h transposed (Gemm1Params).
__global__ __launch_bounds__(THREADS, PP_WAVES_PER_SIMD) void gemm1_big_train_kernel(Gemm1Params<bf16_t> p) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[PP_SMEM];
    big_tile<true, 1>(p, Gemm2Params<bf16_t>{}, smem);
}

// The gate/up GEMM of the masked layer's training forward: the same tiles,
// plus g and u of every row (Gemm1Params).
__global__ __launch_bounds__(THREADS, PP_WAVES_PER_SIMD) void gemm1_big_train_rm_kernel(Gemm1Params<bf16_t> p) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[PP_SMEM];
    big_tile<true, 2>(p, Gemm2Params<bf16_t>{}, smem);
}

__global__ __launch_bounds__(THREADS, PP_WAVES_PER_SIMD) void gemm2_big_kernel(Gemm2Params<bf16_t> p) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[PP_SMEM];
    big_tile<false>(Gemm1Params<bf16_t>{}, p, smem);
}

hipError_t launch_gemm1_big(const Gemm1Params<bf16_t>& p, int grid, hipStream_t s, bool alone) {
    if (grid <= 0) return hipSuccess;
    const int xg = alone ? 32 : XCD_GROUP;
    const int g = (grid + 8 * xg - 1) / (8 * xg) * (8 * xg);
    if (alone) gemm1_big_kernel<32><<<g, THREADS, 0, s>>>(p);
    else gemm1_big_kernel<XCD_GROUP><<<g, THREADS, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_gemm1_big_train(const Gemm1Params<bf16_t>& p, int grid, hipStream_t s) {
    if (grid <= 0) return hipSuccess;
    const int g = (grid + 8 * XCD_GROUP - 1) / (8 * XCD_GROUP) * (8 * XCD_GROUP);
    gemm1_big_train_kernel<<<g, THREADS, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_gemm1_big_train_rm(const Gemm1Params<bf16_t>& p, int grid, hipStream_t s) {
    if (grid <= 0) return hipSuccess;
    const int g = (grid + 8 * XCD_GROUP - 1) / (8 * XCD_GROUP) * (8 * XCD_GROUP);
    gemm1_big_train_rm_kernel<<<g, THREADS, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_gemm2_big(const Gemm2Params<bf16_t>& p, int grid, hipStream_t s) {
    if (grid <= 0) return hipSuccess;
    const int g = (grid + 8 * XCD_GROUP - 1) / (8 * XCD_GROUP) * (8 * XCD_GROUP);
    gemm2_big_kernel<<<g, THREADS, 0, s>>>(p);
    return hipGetLastError();
}

}  // namespace flexmoe
