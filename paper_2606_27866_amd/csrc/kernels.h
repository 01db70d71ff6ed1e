// Kernel declarations and argument blocks of the FlexMoE HIP library.
#pragma once

#include <type_traits>

#include "common.h"

namespace flexmoe {

struct KeepArgs {
    int32_t v[kMaxExperts];
};

// Which segments one GEMM launch covers.  The shared expert needs no routing,
// so its GEMMs can run on a second stream while the routed experts are being
// dispatched; each launch then covers one part of the tile list.
enum GemmPart : int32_t {
    kPartRange = 0,   // segments [seg_lo, seg_hi) (tiles tstart[seg_lo] .. tstart[seg_hi])
    kPartShared = 1   // the shared expert alone; its tile count comes from the host
};

// Gate/up GEMM with fused SwiGLU:
//   H[row][c] = silu(<W_gate[c], x_t>) * <W_up[c], x_t>,  c < k_s
// over every segment s (routed experts, then the shared expert).
template <typename T>
struct Gemm1Params {
    const T* x;                 // [T][d]
    const T* wg;                // routed gate [E][I][d]
    const T* wu;                // routed up   [E][I][d]
    const T* sg;                // shared gate [I_s][d]
    const T* su;                // shared up   [I_s][d]
    const int32_t* perm;        // grouped row -> assignment id
    const SegMeta* seg;         // [nseg]
    const int32_t* tstart;      // [nseg+1] first tile of each segment
    T* H;                       // routed activations [A][I]
    T* Hs;                      // shared activations [T][I_s]
    int d, I, Is, E, top_k, nseg, tokens;
    int part;                   // GemmPart
    int seg_lo, seg_hi;         // kPartRange: the segments covered
    int shared_tiles;           // tiles of the shared segment (kPartShared)
    int clipped;                // routed weights in the clipped layout (see RoutedWeights)
    // Training forwards: g and u for every channel the GEMM computes (c < kg),
    // in the fragment-blocked layout (common.h) of a routed [A][I] and a shared
    // [T][I_s] matrix (launch_gemm1_big_train: routed rows only;
    // launch_gemm1_big_train_rm: all rows).
    T* G;
    T* U;
    T* Gs;
    T* Us;
    // fp32 matrix-core tiles: rows per tile (32, 64 or 128)
    int bm;
    // launch_gemm1_big_train only: the routed rows' activations h transposed --
    // element [c][prow0 + r] for row r of a segment -- with zeros in the rows
    // [rows, packed_width(rows)) of each segment; rows from there to the next
    // segment are neither written nor read.  Row stride ldt.
    T* ht;
    int ldt;
    int nt_all;  // 128 x 128 tiles: see mid_nt_all
};

// Down GEMM: O[row][n] = sum_{c < k_s} H[row][c] * W_down[n][c].  O holds one
// row per routed assignment (and per token for the shared expert); it is fp32
// in fp32 mode and bf16 (rounded once from the fp32 sum) in bf16 mode.
template <typename T>
struct Gemm2Params {
    typedef typename std::conditional<std::is_same<T, float>::value, float, bf16_t>::type OT;
    const T* H;
    const T* Hs;
    const T* wd;                // routed down [E][d][I]
    const T* sd;                // shared down [d][I_s]
    const SegMeta* seg;
    const int32_t* tstart;
    OT* O;                      // routed rows [A][d]
    OT* Os;                     // shared rows [T][d] (split reductions: [splits][T][d])
    int d, I, Is, E, nseg, tokens;
    int ks2;                    // > 0: the shared reduction is split into chunks of ks2 channels
    int part;                   // GemmPart
    int seg_lo, seg_hi;         // kPartRange: the segments covered
    int shared_tiles;           // tiles of the shared segment (kPartShared)
    int clipped;                // routed weights in the clipped layout (see RoutedWeights)
    // Tile order (kPartRange): tstart, seg_lo and seg_hi count positions in
    // this order of the segments (NULL: segment order).  The dispatch puts the
    // shared expert first, then the routed experts by decreasing GEMM width:
    // the longest reductions start first, so the launch ends evenly.
    const int32_t* order = nullptr;
    int bm = 0;                 // fp32 matrix-core tiles: rows per tile
    // training forward (prefill tiles): reduce over the kept channels kk, not
    // over the GEMM width kg, which is I there
    int kept_only = 0;
    int nt_all = 0;             // 128 x 128 tiles: see mid_nt_all
};

// Where routed expert e's weights live.  Ranked layout (online clipping):
// gate/up [E][I][d], down [E][d][I]; expert e's blocks start at e*I*d and a
// down row holds I channels.  Clipped layout (one budget exported offline):
// the experts' blocks are packed back to back, expert e holding
// packed_width(k_e) channels -- gate/up [kp_e][d], down [d][kp_e] -- from
// packed channel ch0; both blocks start at ch0*d and a down row holds kp_e
// channels.
struct RoutedWeights {
    size_t base;   // element offset of the expert's gate/up block and of its down block
    int rows;      // gate/up rows the block holds
    int ldd;       // elements per down row
};
template <typename P>
__device__ __forceinline__ RoutedWeights routed_weights(const P& p, const SegMeta& sm) {
    if (p.clipped) return RoutedWeights{(size_t)sm.ch0 * p.d, packed_width(sm.kk), packed_width(sm.kk)};
    return RoutedWeights{(size_t)sm.e * p.I * p.d, p.I, p.I};
}

// Segment at tile-order position i (down GEMM: Gemm2Params::order).
__device__ __forceinline__ int order_of(const Gemm1Params<bf16_t>&, int i) { return i; }
__device__ __forceinline__ int order_of(const Gemm1Params<float>&, int i) { return i; }
template <typename T>
__device__ __forceinline__ int order_of(const Gemm2Params<T>& p, int i) {
    return p.order ? min(max(p.order[i], 0), p.nseg - 1) : i;
}

// Tile L of a launch -> segment s, its metadata and the tile's index inside
// the segment.  False when L is past the launch's last tile (the caller's
// workgroup then has nothing to do).  The shared segment's metadata is known
// without the dispatch tables: rows = tokens, channels = I_s.  The shared
// expert, when present, is always segment 0.
template <typename P>
__device__ __forceinline__ bool tile_of(const P& p, int L, int& s, SegMeta& sm, int& local) {
    if (p.part == kPartShared) {
        if (L >= p.shared_tiles) return false;
        // the argument values are pinned in scalar registers here: otherwise
        // the compiler may merge the read of `tokens` with the routed path's
        // read of seg[s].rows into one generic (flat) load, one more memory
        // round trip at the start of every tile
        int tokens = p.tokens, is = p.Is;
        asm volatile("" : "+s"(tokens), "+s"(is));
        s = 0;
        sm = SegMeta{0, tokens, is, 0, is, -1, 0, 0};
        local = L;
        return true;
    }
    const int t_lo = p.tstart[p.seg_lo], t_hi = p.tstart[p.seg_hi];  // both requested before either is used
    L += t_lo;
    if (L >= t_hi) return false;
    const int i = find_segment(p.tstart, p.nseg, L);
    s = order_of(p, i);
    sm = p.seg[s];
    local = L - p.tstart[i];
    return true;
}

// Tile shapes of the kernel families (the dispatch kernel builds tile tables
// with these numbers).
constexpr int kF32BM = 64, kF32BN = 64;                      // fp32 on the vector ALUs
// fp32 on the matrix cores: at most kF32MBM rows (f32_rows_per_tile)
constexpr int kF32MBM = 128, kF32MBN1 = 64, kF32MBN2 = 128;
// Whether an fp32 forward of T tokens takes the matrix-core tiles: every
// operand block one tile addresses must stay below 2^31 bytes (32-bit buffer
// offsets); there is no other limit, and no size at which the vector-ALU
// tiles were faster.
inline bool f32_matrix_tiles(long long T, long long d, long long I, long long Is) {
    const long long w = d > (I > Is ? I : Is) ? d : (I > Is ? I : Is), n = I > Is ? I : Is;
    return T * w < (1LL << 29) && n * d < (1LL << 29);
}
constexpr int kBigBM1 = 256, kBigBN1 = 128, kBigBM2 = 256, kBigBN2 = 256;
constexpr int kMidBM = 128, kMidBN1 = 64, kMidBN2 = 128;
constexpr int kDecodeMaxT = 64;     // T at or below which the weight-streaming kernels run
constexpr int kGemvMaxT = 8;        // T at or below which the routed experts' weight-streaming
                                    // GEMMs run on the vector ALUs, in tiles of kDecBN channels /
                                    // output columns (launch_gemm*_decode); above, in tiles of
                                    // kDecWideBN on the matrix cores (launch_gemm*_decode_wide)
constexpr int kDecBN = 16;
constexpr int kDecWideBN = 64;
constexpr int kDecodeWideSharedT = 5;  // above this many tokens the shared expert takes the wide
                                       // tiles too
constexpr int kSharedSplit2T = 16;  // above this many (decode) tokens the shared expert's down
                                    // reduction is split into chunks of 2 I channels, else of I

// Whether the routed experts of a bf16 forward of T > kDecodeMaxT tokens take
// the 128 x 128 tiles (gemm_mid.hip) rather than the 256 x 256 ones, from the
// mean rows of an expert, n = T top_k / E:
//   n <= kMidRows: streaming weights bounds the layer (at 60 % of the channels,
//     small against large tiles: Qwen2-57B shape, n = 10 / 38 / 48, 420 / 529 /
//     562 us against 491 / 585 / 602; n = 75: 695 against 678);
//   n <= kMidRowsFew while the large tiles of the full width would number
//     fewer than kMidWaves per compute unit, so that their last wave is a large
//     part of the launch (Qwen1.5-MoE shape, n = 68 / 100: 215 / 266 us against
//     242 / 308; Mixtral shape, n = 100: 437 against 512; past that, n = 137
//     and 150, the two are equal);
//   but no more than kMidRowsFull where the large tiles of the full width have
//     no such wave: without a shared expert, whose tiles fill it too, and with
//     both GEMMs' tiles filling 7/8 of their waves, each weighted with its
//     reduction, and reductions of kMidFullK on average, beside which a tile's
//     prologue and epilogue are short.  At n = 125 and all channels, small
//     against large: 8 experts of 8192 channels, hidden size 8192, 691 / 584 us;
//     16 of 4096, 4096, 363 / 333; 64 of 1536, 4096, 554 / 513; 24 of 2560, 5120,
//     467 / 404; 32 of 2048, 3072, 297 / 292 (at 60 % 474 / 476, 292 / 305 (70 %),
//     408 / 401, 340 / 345, 221 / 234).  Where one of the three does not hold:
//     waves 3/4 full, 16 of 3072, 3072, 238 / 237 (n = 102: 220 / 227); short
//     reductions, 32 of 2048, 2048, 211 / 233; the 16 of 4096 beside a shared
//     expert of 4096 channels, 443 / 449.  At n = 75 to 87 the small tiles are at
//     worst 2 % behind (8 of 8192 at n = 75: 516 / 555).
constexpr int kMidRows = 48, kMidRowsFew = 128, kMidWaves = 4, kMidRowsFull = 96, kMidFullK = 2304;
inline bool mid_tiles(int T, int top_k, int E, int I, int d, bool has_shared, int compute_units) {
    const long long A = (long long)T * top_k, cu = compute_units;
    if (A <= (long long)kMidRows * E) return true;
    const long long n1 = (long long)E * ceil_div(I, kBigBN1), n2 = (long long)E * ceil_div(d, kBigBN2);
    if (A > (long long)kMidRowsFew * E || n1 >= kMidWaves * cu) return false;
    if (A <= (long long)kMidRowsFull * E || has_shared) return true;
    const long long waves1 = (n1 + cu - 1) / cu, waves2 = (n2 + cu - 1) / cu, k = waves1 * d + waves2 * I;
    return 8 * (n1 * d + n2 * I) < 7 * k * cu || k < kMidFullK * (waves1 + waves2);
}

// Whether the shared expert's tiles may be 128 x 128 ones, which they are where
// one launch covers it and routed experts that take them (no side stream).  Its
// work bounds such a launch once it is large, and where its weight rows start
// inside cache lines (128 bytes), every row piece a tile reads spans one line
// more: small tiles read more of them for their flops.  No-allocation forward,
// the weights of three and more layers in turn, small against large tiles: 49
// shapes without whole lines and with 50 GFLOP or more, 6 % slower on average
// (hidden size 1840, 29 experts of 328 channels, shared 8560, 572 tokens, 54
// GFLOP: 136 / 106 us; 1528, 53 of 1128, 6104, 1299, 73: 188 / 169); at 40 to 50
// GFLOP 2 % faster, below 30 19 %; with whole lines 2 % faster from 50 on.
constexpr double kMidSharedFlops = 50e9;
inline bool mid_one_launch(int T, int d, int I_shared) {
    return ((d | I_shared) & 63) == 0 || 6.0 * T * d * I_shared < kMidSharedFlops;
}

// Whether the 128 x 128 tiles read weights that one row tile uses with the
// non-temporal hint even if their rows start inside 128-byte lines.  Such rows
// are read faster without it (gemm_mid.hip), but plain reads of all routed
// weights crowd out the operands of a shared expert on the side stream, whose
// few large tiles then set the end.  So beside a side stream: while the routed
// weights (6 E I d bytes at 5 TB/s) take less time than the shared expert's two
// reductions, one tile after the other (1.5 us per K tile of 64, half as much
// again beside the routed reads; the down one split from 1024 channels on).
// With the hint / without, top-4, 60 % of the channels, the weights of several
// layers in turn: hidden size 3656, 51 experts of 328 and of 648 channels, shared
// 1320, 248 tokens 139 / 181 and 176 / 207 us; past the line 3664, 30 of 2024,
// 1040, 127 tokens 249 / 226; 1144, 61 of 968, 488, 144 tokens 96 / 88; 1200, 94
// of 832, 552, 807 tokens 131 / 126.  (One layer repeated, its weights in the
// last-level cache, loses more by the hint: the last two 117 / 99 and 99 / 86.)
inline bool mid_nt_all(int E, int I, int d, int I_shared) {
    const double routed_us = 6.0 * E * I * d / 5e6;
    const double shared_us = 1.5 * 1.5 * (d + (I_shared < 1024 ? I_shared : 1024)) / 64;
    return routed_us < shared_us;
}

__global__ void route_kernel(const float* logits, int T, int E, int k, int norm_topk, int32_t* idx,
                             float* wts, int32_t* blockcnt, int NB);
__global__ void dispatch_scan_kernel(const int32_t* blockcnt, int NB, int32_t* blockbase,
                                     int32_t* counts);
// `packed_limit`: in the clipped layout, the packed channels the weight
// buffers hold; an expert whose block would reach past it is treated as
// k_e = 0 (the ranked layout passes INT32_MAX).  `plan` (NULL: experts in id
// order, GEMM width = k_e): the bucketed forward's segment order plan[0..E)
// (expert ids) and GEMM widths plan[E..2E).
// keep = NULL: the plan alone
__global__ void set_plan_kernel(int32_t* keep, int32_t* plan, KeepArgs k, KeepArgs order, KeepArgs kg, int E);
__global__ void dispatch_scatter_kernel(const int32_t* idx, const int32_t* keep,
                                        const int32_t* counts, const int32_t* blockbase, int T,
                                        int E, int k, int I, int I_shared, int d, int NB,
                                        TileShape ts, int packed_limit, const int32_t* plan,
                                        int32_t* perm, int32_t* pos,
                                        int32_t* offsets, SegMeta* seg, int32_t* t1start,
                                        int32_t* t2start, int32_t* order2);
hipError_t launch_dispatch_small(const float* logits, int T, int E, int k, int norm_topk, const int32_t* keep, int I,
                                 int I_shared, int d, TileShape ts, int packed_limit, const int32_t* plan,
                                 int pre_routed, int32_t* idx, float* wts, int32_t* counts, int32_t* perm,
                                 int32_t* pos, int32_t* offsets, SegMeta* seg, int32_t* t1start, int32_t* t2start,
                                 int32_t* order2, hipStream_t s);
__global__ void set_keep_kernel(int32_t* keep, KeepArgs t, int E);

// Rows per fp32 matrix-core tile of a GEMM with `cols` column tiles: halved
// from 128 to at least 32 while the segment with the most rows (the shared
// expert's T, else the mean of the routed ones, all together) has fewer tiles
// than the chip has compute units.  Its tiles are the longest of the launch: a
// shared down projection of 500 rows and 5632 channels in 64 tiles took 420
// us, in 256 tiles 247.
inline int f32_rows_per_tile(int T, int E, int top_k, bool has_shared, int cols, int compute_units) {
    const long long rows = has_shared ? T : ((long long)T * top_k + E - 1) / E, segs = has_shared ? 1 : E;
    int bm = kF32MBM;
    while (bm > 32 && segs * ((rows + bm - 1) / bm) * cols < compute_units) bm /= 2;
    return bm;
}

// Launchers (defined next to their kernels).  Each returns the launch status.
// alone (gate/up): no side-stream launch runs beside it.
hipError_t launch_gemm1_big(const Gemm1Params<bf16_t>& p, int grid, hipStream_t s, bool alone);
hipError_t launch_gemm2_big(const Gemm2Params<bf16_t>& p, int grid, hipStream_t s);
// Between decode and prefill (mid_tiles): 128 x 128 tiles, two workgroups per
// compute unit (gemm_mid.hip).
hipError_t launch_gemm1_mid(const Gemm1Params<bf16_t>& p, int grid, hipStream_t s);
hipError_t launch_gemm2_mid(const Gemm2Params<bf16_t>& p, int grid, hipStream_t s);
// T <= kGemvMaxT: 16-wide tiles on the vector ALUs (gemv_decode.hip).
hipError_t launch_gemm1_decode(const Gemm1Params<bf16_t>& p, int tiles, hipStream_t s);
hipError_t launch_gemm2_decode(const Gemm2Params<bf16_t>& p, int tiles, hipStream_t s);
// T <= kDecodeMaxT: tiles of kDecWideBN channels / output columns on the
// matrix cores (gemm_decode.hip).
hipError_t launch_gemm1_decode_wide(const Gemm1Params<bf16_t>& p, int tiles, hipStream_t s);
hipError_t launch_gemm2_decode_wide(const Gemm2Params<bf16_t>& p, int tiles, hipStream_t s);
// matrix: f32_matrix_tiles, else 64 x 64 tiles on the vector ALUs.
hipError_t launch_gemm1_f32(const Gemm1Params<float>& p, int grid, hipStream_t s, bool matrix);
hipError_t launch_gemm2_f32(const Gemm2Params<float>& p, int grid, hipStream_t s, bool matrix);
hipError_t launch_combine(const void* O, const void* Os, const int32_t* pos, const float* wts,
                          int T, int k, int d, int shared_parts, int dtype, void* y, hipStream_t s);
hipError_t launch_rank_reorder(const float* scores, const void* wg, const void* wu,
                               const void* wd, void* wg_r, void* wu_r, void* wd_r,
                               int32_t* perm, int E, int I, int d, int esize, hipStream_t s);
// Packs one budget's ranked weights into the clipped layout (RoutedWeights);
// keep holds the budget, already validated on the host.
hipError_t launch_export_clipped(const KeepArgs& keep, const void* wg_r, const void* wu_r,
                                 const void* wd_r, void* wg_c, void* wu_c, void* wd_c, int E, int I,
                                 int d, int esize, hipStream_t s);

}  // namespace flexmoe
