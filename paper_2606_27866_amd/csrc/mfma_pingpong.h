// K loop of the 256 x 256 bf16 MFMA tiles (gfx950), shared by the prefill
// GEMMs, the training backward and the saliency's weight gradients.
//
// C[m][n] = sum_k A[m][k] B[n][k] for one workgroup of 8 waves, both operands
// contiguous in K.  Wave (wm, wn) = (wave / 4, wave % 4) owns, in each of the
// four 128 x 128 quadrants (A half ah, B half bh), 16*MF rows of A and 32
// rows of B as v_mfma_f32_16x16x32_bf16 accumulators (128 registers at
// MF = 4).
//
// Ping-pong: waves w and w + 4 share a SIMD and run half a phase apart (the
// wm = 1 waves take one extra barrier at the start), so that on every SIMD
// one wave multiplies a quadrant (16 MFMAs, the matrix core's alone) while
// the other reads its next fragments from LDS and requests operands from
// memory; an s_barrier after each of the two parts swaps them.  A K tile of
// 64 takes four phases:
//   phase   LDS reads            requests from memory   multiplies
//     0     A half 0 (tile kt)   A half 1 (kt + 1)      A0 x B0
//     1     B half 1 (kt)        B half 0 (kt + 2)      A0 x B1
//     2     A half 1 (kt)        A half 0 (kt + 2)      A1 x B1
//     3     B half 0 (kt + 1)    B half 1 (kt + 2)      A1 x B0
// Every phase reads one 16 KB half from LDS and requests one (buffer_load ...
// lds, two instructions per wave), so the LDS and the address units see an
// even load, where requesting a K tile at one point stalled the MFMAs behind
// a burst of 64 requests.  LDS holds two K tiles (128 KB).  A half read in
// phase i is refilled from phase i + 2 on: every wave's reads of it are done
// by the end of the slot in which the lagging waves multiply phase i, one
// barrier before.  The request leaves six phases (about 3000 clocks) before
// the data is read; the wait at the end of each phase leaves the last five
// phases' requests in flight, and the two barriers that follow publish the
// data to all waves before phase i + 8 reads it.
//
// Dense 16384 x 14336 x 4096, 8192^3 and 16384 x 4096 x 7168 on one MI355X:
// 1418, 1510 and 1460 TFLOP/s, against 1260-1285, 1320 and 1280 for two waves
// per SIMD without the phase shift on 32x32x16 MFMAs (and 1506, 1525, 1528
// for the vendor's dense GEMM).  The same loop on 32x32x16 MFMAs: 1322, 1405
// and 1360: at the power limit the smaller shape runs at a higher clock.
// Waiting for the LDS reads before the barrier instead of after it, or
// leaving the waves' priorities equal, changes nothing measurable.
#pragma once

#include <type_traits>

#include "mfma_tile.h"

namespace flexmoe {
namespace mfma {

constexpr int PP_BM = 256, PP_BN = 256;          // tile
constexpr int PP_WAVES = 8, PP_THREADS = 64 * PP_WAVES;
constexpr int PP_WAVES_PER_SIMD = PP_WAVES / 4;
constexpr int PP_HALF_ROWS = 128;                // LDS rows of an operand half
constexpr int PP_HALF = PP_HALF_ROWS * ROWB;     // 16 KB
constexpr int PP_SMEM = 2 * 4 * PP_HALF;         // two K tiles of [A0 A1 B0 B1]: 128 KB
constexpr int PP_RPI = 64 / CHUNKS;              // LDS rows one DMA instruction fills
constexpr int PP_ND = PP_HALF_ROWS / (PP_WAVES * PP_RPI);  // DMA instructions per wave and half
static_assert(PP_ND == 2, "the waits count two requests per wave and phase");

// Operand rows this lane requests.  DMA instruction i of a wave fills LDS
// rows wave*16 + i*8 .. +8 of a half; lane -> row lane/8, LDS chunk lane%8,
// which holds the row's K chunk swz(row, lane%8).  col[i] is that chunk's
// first K element (the same in both halves of both operands); aoff/boff are
// the byte offsets of K tile 0 (kOOB: the row reads zeros).
struct PPOperands {
    __amdgpu_buffer_rsrc_t ra, rb[2];
    uint32_t aoff[2][PP_ND], boff[2][PP_ND];
    int col[PP_ND];
    int K;
};

// Two pairs of operands with the same rows, offsets, extents (in elements) and
// K: C = A B^T + A2 B2^T, the K tiles of the second pair after those of the
// first (ra and rb of PPOperands are then unused).
struct PPSecond {
    const bf16_t *a, *a2, *b, *b2;
    size_t aext, bext;
};

// LDS row (within a half) and K chunk column of DMA instruction i.
__device__ __forceinline__ int pp_lds_row(int wave, int lane, int i) {
    return wave * (PP_ND * PP_RPI) + i * PP_RPI + lane / CHUNKS;
}
__device__ __forceinline__ int pp_col(int wave, int lane, int i) {
    return swz(pp_lds_row(wave, lane, i), lane % CHUNKS) * 8;
}

// 16-row A fragments per wave and half for a tile of `rows` rows: the two
// halves of 32*mf rows cover them.
__device__ __forceinline__ int pp_mf(int rows) { return min(4, (rows + 63) >> 6); }

// Rows per row tile of a segment of `rows` rows: its ceil(rows / 256) row
// tiles take equal shares, rounded up to the 64-row steps of the MFMA work.
// 273 rows go as 192 + 81 (3 + 2 steps) where 256 + 17 (4 + 1) cost as much
// MFMA work and left one tile twice as long as the rest (a tile's requests,
// prologue and epilogue do not shrink with its rows).
__device__ __forceinline__ int pp_row_step(int rows) {
    const int mt = ceil_div(rows, PP_BM);
    return ceil_div(ceil_div(rows, mt), 64) * 64;
}

// Tile row of LDS row r of A half h (valid below 32*mf).
__device__ __forceinline__ int pp_a_row(int h, int r, int mf) { return h * 32 * mf + r; }

// Accumulators: acc[ah][bh][j * MF + i] is the 16 x 16 product of A fragment
// i and B fragment j of the quadrant.  With kSwap = false the B fragment is
// the MFMA's first operand: lane -> A row lane%16 of the fragment, register v
// -> B row 4*(lane/16) + v (a lane holds runs of 4 consecutive B rows of one
// A row).  kSwap = true exchanges the operands' roles.
template <int MF>
using PPAcc = floatx4[2][2][2 * MF];

// Row of the tile (A side) / column (B side) of fragment i / j in half h,
// before the lane's part.
template <int MF>
__device__ __forceinline__ int pp_frag_row(int h, int wm, int i) { return h * 32 * MF + wm * 16 * MF + i * 16; }
__device__ __forceinline__ int pp_frag_col(int h, int wn, int j) { return h * PP_HALF_ROWS + wn * 32 + j * 16; }

// Tail of a K loop that needs nothing after its last K tile: the requests past
// the end read zeros.
struct PPZeroTail {
    __device__ __forceinline__ void operator()(int, int, unsigned char*) const {}
};

// No second pair.
struct PPNoSecond {};

// Runs the K loop.  Requests for K tiles past the end (slot h = kt - nk is 0
// or 1) go to tail(half, h, dst), half 0..3 = A0 A1 B0 B1, which must issue
// exactly PP_ND loads into this wave's rows `dst` of that half; half 1 (A1)
// of slot 1 is never requested.  On return this wave has no request in flight
// and every wave has finished its LDS reads.
template <int MF, bool kSwap, typename Tail, typename Second = PPNoSecond>
__device__ __forceinline__ void pp_loop(unsigned char* smem, const PPOperands& op, int wave, int lane,
                                        PPAcc<MF>& acc, Tail&& tail, Second sec = Second{}) {
    constexpr bool kTail = !std::is_same<std::decay_t<Tail>, PPZeroTail>::value;
    constexpr bool kSecond = std::is_same<Second, PPSecond>::value;
    const int wm = wave >> 2, wn = wave & 3;
    const int nk1 = ceil_div(op.K, BK), nk = kSecond ? 2 * nk1 : nk1;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int f = 0; f < 2 * MF; ++f) acc[q >> 1][q & 1][f] = floatx4{0.f, 0.f, 0.f, 0.f};
    // half 0: A0, 1: A1, 2: B0, 3: B1
    auto request = [&](int half, int kt, auto may_end) {
        unsigned char* dst = smem + ((kt & 1) * 4 + half) * PP_HALF + wave * (PP_ND * PP_RPI) * ROWB;
        if constexpr (kTail && decltype(may_end)::value)
            if (kt >= nk) {
                tail(half, kt - nk, dst);
                return;
            }
        __amdgpu_buffer_rsrc_t r = half < 2 ? op.ra : op.rb[half & 1];
        if constexpr (kSecond) {
            const bool second = kt >= nk1;
            r = half < 2 ? make_rsrc(second ? sec.a2 : sec.a, sec.aext) : make_rsrc(second ? sec.b2 : sec.b, sec.bext);
            if (second) kt -= nk1;
        }
        // past the end `lim` is not positive: every lane's offset is kOOB, with
        // no branch in the loop (branches around the requests cost 8 % of a
        // dense product)
        const int lim = op.K - kt * BK;
        const uint32_t soff = (uint32_t)(kt * BK) * 2u;
#pragma unroll
        for (int i = 0; i < PP_ND; ++i) {
            const uint32_t o = half < 2 ? op.aoff[half & 1][i] : op.boff[half & 1][i];
            load_lds16(r, op.col[i] < lim ? o : kOOB, soff, dst + i * PP_RPI * ROWB);
        }
    };
    bf16x8 fa[MF][2], fx[2][2], fy[2][2];  // [fragment][32-deep K step]
    const int lr = lane & 15, lc = lane >> 4;
    auto read_a = [&](int half, int kt) {
        const unsigned char* b = smem + ((kt & 1) * 4 + half) * PP_HALF;
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int s = 0; s < 2; ++s) fa[i][s] = lds_frag(b, wm * 16 * MF + i * 16 + lr, s * 4 + lc);
    };
    auto read_b = [&](int half, int kt, bf16x8 (&f)[2][2]) {
        const unsigned char* b = smem + ((kt & 1) * 4 + 2 + half) * PP_HALF;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int s = 0; s < 2; ++s) f[j][s] = lds_frag(b, wn * 32 + j * 16 + lr, s * 4 + lc);
    };
    // the second part of a phase: swap with the other wave of the SIMD,
    // multiply, swap back
    auto multiply = [&](floatx4 (&c)[2 * MF], const bf16x8 (&f)[2][2]) {
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(5 * PP_ND));
        __builtin_amdgcn_sched_barrier(0);
        barrier_no_fence();
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
        __builtin_amdgcn_s_setprio(1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int i = 0; i < MF; ++i)
                    c[j * MF + i] = kSwap ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i][s], f[j][s], c[j * MF + i], 0, 0, 0)
                                          : __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[j][s], fa[i][s], c[j * MF + i], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(0);
        barrier_no_fence();
        __builtin_amdgcn_sched_barrier(0);
    };
    // B half 0 of tile kt is in x at the start; x holds B half 0 and y B half
    // 1 of the tile, and y B half 0 of the next tile at the end
    auto tile = [&](int kt, bf16x8 (&x)[2][2], bf16x8 (&y)[2][2], auto may_end) {
        read_a(0, kt);
        request(1, kt + 1, may_end);
        multiply(acc[0][0], x);
        read_b(1, kt, y);
        request(2, kt + 2, may_end);
        multiply(acc[0][1], y);
        read_a(1, kt);
        request(0, kt + 2, may_end);
        multiply(acc[1][1], y);
        read_b(0, kt + 1, y);
        request(3, kt + 2, may_end);
        multiply(acc[1][0], x);
    };
    constexpr std::true_type end{};
    request(2, 0, end);
    request(0, 0, end);
    request(3, 0, end);
    request(1, 0, end);
    request(2, 1, end);
    request(0, 1, end);
    request(3, 1, end);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(5 * PP_ND));  // B0 and A0 of tile 0 are in
    barrier_no_fence();
    if (wm == 1) barrier_no_fence();  // the lagging waves; the leading ones wait at the end
    __builtin_amdgcn_sched_barrier(0);
    read_b(0, 0, fx);
    int kt = 0;
    if constexpr (kTail)  // the pairs of tiles whose requests stay before the end
        for (; kt + 3 < nk; kt += 2) {
            tile(kt, fx, fy, std::false_type{});
            tile(kt + 1, fy, fx, std::false_type{});
        }
    for (; kt + 1 < nk; kt += 2) {
        tile(kt, fx, fy, end);
        tile(kt + 1, fy, fx, end);
    }
    if (kt < nk) tile(kt, fx, fy, end);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0) & kWaitLgkm0);
    if (wm == 0) barrier_no_fence();
    __builtin_amdgcn_sched_barrier(0);
}

// Runs `body` with the fragment count of a tile of `rows` rows.
template <typename F>
__device__ __forceinline__ void pp_by_rows(int rows, F&& body) {
    switch (pp_mf(rows)) {
        case 4: body(std::integral_constant<int, 4>{}); break;
        case 3: body(std::integral_constant<int, 3>{}); break;
        case 2: body(std::integral_constant<int, 2>{}); break;
        default: body(std::integral_constant<int, 1>{}); break;
    }
}

}  // namespace mfma
}  // namespace flexmoe
