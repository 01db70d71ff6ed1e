// Ragged grouped GEMMs on bf16 MFMA for batches between decode and prefill:
// more than kDecodeMaxT tokens, but few rows per routed expert (mid_tiles in
// kernels.h).
//
// A routed expert then holds some tens of rows, and the layer is bound by
// streaming its weights (Eq. 4: the first k_e channels) while the shared
// expert, which sees every token, is bound by the matrix cores.  The 256 x 256
// tiles of gemm_bf16_big.hip take a whole compute unit each: a 40-row expert
// leaves most of it idle, and the two kinds of tile cannot share one.  Here a
// workgroup of 4 waves owns a tile of 128 rows x 128 weight rows (64 channels'
// gate and up rows, or 128 output columns) in 80 KB of LDS and under 256
// VGPRs, so that two run on every compute unit and one's waits for memory are
// covered by the other's MFMAs.
//   - K tiles of 64 as in mfma_tile.h (128-byte LDS rows, XOR-swizzled 16-byte
//     chunks, buffer_load ... lds).  The weights are requested two K tiles
//     ahead (three stages of 16 KB, 64 KB in flight per compute unit); the
//     token rows, which the L2 holds, one ahead (two stages of 16 KB) or, in a
//     tile of at most 64 rows, two ahead (three of 8 KB).
//   - one barrier per K tile: it publishes the tile's operands and frees the
//     stages of the tile before it.
//   - wave (wm, wn) = (wave / 2, wave % 2) multiplies 16*MF rows (MF = 1..4,
//     so the MFMA work follows the rows in steps of 32) by 64 weight rows;
//     gate and up of a channel sit in the same lane.
// At 60 % of the channels, 256 x 256 tiles -> these: Qwen2-57B shape at 80 and
// 300 tokens 491 -> 420 and 585 -> 529 us, Qwen1.5-MoE shape at 100, 300 and
// 1023 159 -> 136, 187 -> 153 and 242 -> 215, Mixtral shape at 80, 200 and 400
// 455 -> 336, 493 -> 364 and 512 -> 437.
#include <type_traits>

#include "mfma_tile.h"

namespace flexmoe {

namespace {
using namespace mfma;
constexpr int MBM = kMidBM, MBN = 128;      // rows x weight rows
constexpr int MWAVES = 4, MTHREADS = 64 * MWAVES;
constexpr int MRPI = 64 / CHUNKS;           // LDS rows one DMA instruction fills
constexpr int MNB = MBN / (MWAVES * MRPI);  // weight DMA instructions per wave and K tile
constexpr int MB_STAGE = MBN * ROWB;        // 16 KB
constexpr int MB_STAGES = 3;
constexpr int MA_BYTES = 2 * MBM * ROWB;    // 32 KB: two stages of 128 rows or three of 64
constexpr int MID_SMEM = MB_STAGES * MB_STAGE + MA_BYTES;
static_assert(2 * MID_SMEM <= 160 * 1024, "two workgroups share a compute unit's LDS");
constexpr int kNonTemporal = 2;             // cache-policy operand of a buffer load
constexpr int MXCD = 8;                     // consecutive tiles kept on one XCD
static_assert(kMidBN1 * 2 == MBN && kMidBN2 == MBN, "the tile tables are built with these widths");
}  // namespace

template <bool kGateUp>
__device__ __forceinline__ void mid_tile(const Gemm1Params<bf16_t>& p1, const Gemm2Params<bf16_t>& p2,
                                         unsigned char* smem) {
    const int d = kGateUp ? p1.d : p2.d;
    const int jb = blockIdx.x >> 3;
    const int L = (jb / MXCD) * (8 * MXCD) + (blockIdx.x & 7) * MXCD + jb % MXCD;
    int s, local;
    SegMeta sm;
    if (!(kGateUp ? tile_of(p1, L, s, sm, local) : tile_of(p2, L, s, sm, local))) return;  // workgroup-uniform
    const bool shared = sm.e < 0;
    // a segment's tiles: row tiles fastest (they share a weight panel through
    // the XCD's L2), then columns; the shared expert's split down reduction
    // has one such grid per chunk
    const int mt = ceil_div(sm.rows, MBM);
    const int nt = kGateUp ? ceil_div(sm.kg, kMidBN1) : ceil_div(d, MBN);
    const int split = kGateUp ? 0 : local / (mt * nt);
    const int loc = local - split * mt * nt;
    const int ntile = loc / mt, mtile = loc - ntile * mt;
    const int row0 = mtile * MBM, tile_rows = min(MBM, sm.rows - row0);

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int wm = wave >> 1, wn = wave & 1;

    // ---- operands: K range, buffer descriptors, row strides
    int K, lda, ldw;
    uintptr_t wbits;  // the weight rows' first addresses and stride: their low bits
    __amdgpu_buffer_rsrc_t ra, rb;
    if constexpr (kGateUp) {
        K = lda = ldw = d;
        const RoutedWeights rw = shared ? RoutedWeights{0, p1.Is, 0} : routed_weights(p1, sm);
        // waves 0 and 1 request the gate rows, waves 2 and 3 the up rows
        const bf16_t* Wg = (shared ? p1.sg : p1.wg) + rw.base;
        const bf16_t* Wu = (shared ? p1.su : p1.wu) + rw.base;
        wbits = (uintptr_t)Wg | (uintptr_t)Wu;
        ra = make_rsrc(p1.x, (size_t)p1.tokens * d);
        rb = make_rsrc(wave < MWAVES / 2 ? Wg : Wu, (size_t)rw.rows * d);
    } else {
        const bool chunked = shared && p2.ks2 > 0;
        const int kbeg = chunked ? split * p2.ks2 : 0;
        K = chunked ? min(sm.kg - kbeg, p2.ks2) : sm.kg;
        const RoutedWeights rw = shared ? RoutedWeights{0, 0, p2.Is} : routed_weights(p2, sm);
        lda = shared ? p2.Is : p2.I;
        ldw = rw.ldd;
        const bf16_t* Hb = (shared ? p2.Hs : p2.H + (size_t)sm.row0 * p2.I) + kbeg;
        const bf16_t* Wd = (shared ? p2.sd : p2.wd + rw.base) + kbeg;
        wbits = (uintptr_t)Wd;
        ra = make_rsrc(Hb, (size_t)(shared ? p2.tokens : sm.rows) * lda - kbeg);
        rb = make_rsrc(Wd, (size_t)d * ldw - kbeg);
    }
    // DMA instruction i of a wave fills 8 LDS rows; lane -> row lane/8, LDS
    // chunk lane%8, which holds the row's K chunk swz(row, lane%8).  The
    // swizzle uses row bits 1..3 only: the chunk column depends on the parity
    // of i alone.  Masked rows read zeros.
    uint32_t boff[MNB];
    int col[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) col[i] = swz(i * MRPI + lane / CHUNKS, lane % CHUNKS) * 8;
#pragma unroll
    for (int i = 0; i < MNB; ++i) {
        const int r = wave * (MNB * MRPI) + i * MRPI + lane / CHUNKS;
        const int n = kGateUp ? ntile * kMidBN1 + (r & (kMidBN1 - 1)) : ntile * MBN + r;
        const int lim = kGateUp ? sm.kg : d;
        boff[i] = n < lim ? (uint32_t)(((size_t)n * ldw + col[i & 1]) * 2) : kOOB;
    }

    const int nk = ceil_div(K, BK);
    const int lr = lane & 15, lc = lane >> 4;

    // The K loop and epilogue for a tile whose waves hold MF 16-row fragments:
    // wave row wm covers rows wm*16*MF .. of the tile.  kOnce: the segment has
    // one row tile, so its weights are read once and carry the non-temporal
    // hint (Qwen2-57B shape at 80 and 300 tokens 462 -> 420 and 563 -> 529 us,
    // Qwen1.5-MoE shape at 100 and 300 154 -> 136 and 172 -> 153; also on
    // weights that a second row tile reads again, Mixtral shape at 400 tokens,
    // 446 -> 487 against 437 without).  Not on rows that start inside a 128-byte
    // line: a K tile then shares its lines with the next, and the hint has them
    // fetched twice (top-4, hidden size 1072, 35 experts of 1096 channels at 268
    // tokens 72.4 us with it, 70.9 without; 568, 58 of 1952 at 492 97.7 / 93.7;
    // where the weights stay in the last-level cache 99 / 71 and 86.5 / 67.3) --
    // except beside a shared expert that ends later (mid_nt_all).
    auto run = [&](auto mf_tag, auto once_tag) {
        constexpr int MF = decltype(mf_tag)::value;
        constexpr bool kOnce = decltype(once_tag)::value;
        constexpr int AROWS = MF > 2 ? 128 : 64;           // staged token rows
        constexpr int DA = MF > 2 ? 1 : 2;                 // K tiles the token rows are requested ahead
        constexpr int NA = AROWS / (MWAVES * MRPI);        // token-row DMA instructions per wave and K tile
        constexpr int A_STAGE = AROWS * ROWB;
        static_assert((DA + 1) * A_STAGE <= MA_BYTES, "the token-row stages fit");
        unsigned char* sA = smem + MB_STAGES * MB_STAGE;
        uint32_t aoff[NA];
        int src[NA];
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            src[i] = row0 + wave * (NA * MRPI) + i * MRPI + lane / CHUNKS;
            // every lane loads its rows' permutation entries (rows past the
            // segment read its last row's, unused): all requested together
            if (kGateUp && !shared) src[i] = p1.perm[sm.row0 + min(src[i], sm.rows - 1)];
        }
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int r = wave * (NA * MRPI) + i * MRPI + lane / CHUNKS;
            if (kGateUp && !shared) src[i] = (int)min((unsigned)(src[i] / p1.top_k), (unsigned)(p1.tokens - 1));
            aoff[i] = r < tile_rows ? (uint32_t)(((size_t)src[i] * lda + col[i & 1]) * 2) : kOOB;
        }
        // past the end every lane's offset is kOOB: the count of outstanding
        // requests stays exact
        auto request_a = [&](int kt, int stage) {
            const int lim = K - kt * BK;
#pragma unroll
            for (int i = 0; i < NA; ++i)
                load_lds16(ra, col[i & 1] < lim ? aoff[i] : kOOB, (uint32_t)(kt * BK) * 2u,
                           sA + stage * A_STAGE + (wave * NA + i) * (MRPI * ROWB));
        };
        auto request_b = [&](int kt, int stage) {
            const int lim = K - kt * BK;
#pragma unroll
            for (int i = 0; i < MNB; ++i)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    rb, (lds_ptr_t*)(smem + stage * MB_STAGE + (wave * MNB + i) * (MRPI * ROWB)), 16,
                    col[i & 1] < lim ? boff[i] : kOOB, (uint32_t)(kt * BK) * 2u, 0, kOnce ? kNonTemporal : 0);
        };
        floatx4 acc[4][MF];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < MF; ++i) acc[j][i] = floatx4{0.f, 0.f, 0.f, 0.f};
        // weight row of fragment j: gate rows then the same channels' up rows,
        // or 64 output columns
        auto brow = [&](int j) {
            return kGateUp ? (j >> 1) * kMidBN1 + wn * 32 + (j & 1) * 16 : wn * 64 + j * 16;
        };
        request_a(0, 0);
        request_b(0, 0);
        if constexpr (DA == 2) request_a(1, 1);
        request_b(1, 1);
        int sa = 0, sb = 0;  // stages of tile kt
        for (int kt = 0; kt < nk; ++kt) {
            // tile kt is in when only the requests of tile kt + 1 are
            // outstanding; this wave's LDS reads of tile kt - 1 are done, so
            // after the barrier its stages may be refilled
            __builtin_amdgcn_s_waitcnt(waitcnt_vm(DA == 2 ? NA + MNB : MNB) & kWaitLgkm0);
            barrier_no_fence();
            const int ea = sa == 0 ? DA : sa - 1, eb = sb == 0 ? MB_STAGES - 1 : sb - 1;
            request_a(kt + DA, ea);
            request_b(kt + 2, eb);
            const unsigned char* a = sA + sa * A_STAGE;
            const unsigned char* b = smem + sb * MB_STAGE;
            bf16x8 fa[2][MF], fb[2][4];
#pragma unroll
            for (int st = 0; st < 2; ++st) {
#pragma unroll
                for (int j = 0; j < 4; ++j) fb[st][j] = lds_frag(b, brow(j) + lr, st * 4 + lc);
#pragma unroll
                for (int i = 0; i < MF; ++i) fa[st][i] = lds_frag(a, wm * 16 * MF + i * 16 + lr, st * 4 + lc);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int st = 0; st < 2; ++st)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int i = 0; i < MF; ++i)
                        acc[j][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[st][j], fa[st][i], acc[j][i], 0, 0, 0);
            sa = sa == DA ? 0 : sa + 1;
            sb = sb == MB_STAGES - 1 ? 0 : sb + 1;
        }
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));  // no DMA may outlive the workgroup's LDS

        // lane -> row lane%16 of a fragment, registers -> 4 consecutive weight
        // rows from 4*(lane/16): 8-byte stores
        const int sub = lc * 4;
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            const int row = row0 + wm * 16 * MF + i * 16 + lr;
            if (row >= sm.rows) continue;
            if constexpr (kGateUp) {
                const int ldh = shared ? p1.Is : p1.I;
                bf16_t* hr = (shared ? p1.Hs : p1.H + (size_t)sm.row0 * p1.I) + (size_t)row * ldh;
                // channels from kk to the GEMM width rounded up to 8 are
                // written as zeros (the down GEMM reads whole 16-byte chunks)
                const int kk8 = min((sm.kg + 7) & ~7, ldh);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int ch = ntile * kMidBN1 + wn * 32 + j * 16 + sub;
                    if (ch >= kk8) continue;
                    const floatx4 g = acc[j][i], u = acc[j + 2][i];
                    float h[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) h[v] = ch + v < sm.kk ? silu_fast(g[v]) * u[v] : 0.f;
                    *reinterpret_cast<uint2*>(hr + ch) = make_uint2(pack_bf16x2(h[0], h[1]), pack_bf16x2(h[2], h[3]));
                }
            } else {
                bf16_t* orow = (shared ? p2.Os + (size_t)split * p2.tokens * d : p2.O + (size_t)sm.row0 * d) +
                               (size_t)row * d;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int n = ntile * MBN + brow(j) + sub;
                    if (n >= d) continue;
                    const floatx4 o = acc[j][i];
                    *reinterpret_cast<uint2*>(orow + n) = make_uint2(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]));
                }
            }
        }
    };
    auto by_rows = [&](auto once) {
        if (tile_rows > 96) run(std::integral_constant<int, 4>{}, once);
        else if (tile_rows > 64) run(std::integral_constant<int, 3>{}, once);
        else if (tile_rows > 32) run(std::integral_constant<int, 2>{}, once);
        else run(std::integral_constant<int, 1>{}, once);
    };
    if (mt == 1 && ((kGateUp ? p1.nt_all : p2.nt_all) || ((wbits | (uintptr_t)ldw * 2) & 127) == 0))
        by_rows(std::true_type{});
    else by_rows(std::false_type{});
}

__global__ __launch_bounds__(MTHREADS, 2) void gemm1_mid_kernel(Gemm1Params<bf16_t> p) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[MID_SMEM];
    mid_tile<true>(p, Gemm2Params<bf16_t>{}, smem);
}

__global__ __launch_bounds__(MTHREADS, 2) void gemm2_mid_kernel(Gemm2Params<bf16_t> p) {
    __shared__ __attribute__((aligned(1024))) unsigned char smem[MID_SMEM];
    mid_tile<false>(Gemm1Params<bf16_t>{}, p, smem);
}

hipError_t launch_gemm1_mid(const Gemm1Params<bf16_t>& p, int grid, hipStream_t s) {
    if (grid <= 0) return hipSuccess;
    gemm1_mid_kernel<<<(grid + 8 * MXCD - 1) / (8 * MXCD) * (8 * MXCD), MTHREADS, 0, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_gemm2_mid(const Gemm2Params<bf16_t>& p, int grid, hipStream_t s) {
    if (grid <= 0) return hipSuccess;
    gemm2_mid_kernel<<<(grid + 8 * MXCD - 1) / (8 * MXCD) * (8 * MXCD), MTHREADS, 0, s>>>(p);
    return hipGetLastError();
}

}  // namespace flexmoe
