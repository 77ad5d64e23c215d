// Expert FFN (paper Sec. 2.1: every expert is a two-layer fully connected network)
// as two grouped GEMMs over the expert-major buffer:
//   H  = act(xe . W1[e] + b1[e])      rows of expert e only
//   ye = H . W2[e] + b2[e]
// Row ranges per expert are known only on the device; the kernels take them from a
// table of row tiles (plan_tiles) and the grid is sized for the worst case, surplus
// blocks exit at once.
//
// bf16 layers: both operands are stored with the contraction index contiguous (activations by
// nature, weights after moe_pack_weights), and the weights are fed as the MFMA "A" operand
// so that each lane ends up with four consecutive output columns of one row.
// grouped_gemm_w4_kernel runs 256 x 256 tiles and grouped_gemm_mfma_kernel those of 128 rows, tiles of 256 columns on
// the loop of gemm_w4_run.h, 128 x 128 on that of gemm_w4_body.inc; grouped_gemm_stream_kernel runs decode steps;
// grouped_gemm_staged_kernel, whose operands go through registers, 64 x 256 tiles and operands past 32-bit offsets.  H and
// ye are kept in fp16.
// fp32 layers: grouped_gemm_f32_kernel, on the fp32 matrix instruction.
#include "activation.h"
#include "common.h"
#include <cstdio>

#include <hip/hip_ext.h>

#include <type_traits>

namespace moe {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

// ---------------------------------------------------------------- activations
template <int ACT, bool FAST>
__device__ __forceinline__ float activate(float v)
{
    if constexpr (ACT == MOE_ACT_GELU_ERF) {
        if constexpr (FAST) return gelu_erf_fast(v);
        return 0.5f * v * (1.0f + erff(v * 0.70710678118654752f));
    } else if constexpr (ACT == MOE_ACT_GELU_TANH) {
        if constexpr (FAST) return v * half_one_plus_tanh(v);
        return 0.5f * v * (1.0f + tanhf(0.7978845608028654f * (v + 0.044715f * v * v * v)));
    } else if constexpr (ACT == MOE_ACT_RELU) {
        return fmaxf(v, 0.0f);
    } else {
        return v;
    }
}

// ---------------------------------------------------------------- fp32 GEMM
// C[r, n] = act(sum_k A[r,k] B[e][k,n] + bias[e][n]); B canonical [E, K, N].
// 2 x 2 wavefronts of TM x TN v_mfma_f32_16x16x4_f32 (fp32 products and sums, twice the rate of
// v_fmac), 32-deep stages through a double-buffered LDS tile, PD stages of global loads in flight
// in registers.  A lane reads four consecutive k of a token row at once and feeds them to four
// instructions, the weights one by one at the same four k (no bank conflicts either way).
// Small layers are bound by the latency of a few stages on a few tiles, hence the deep prefetch and
// the 32 x 32 tile (TM = TN = 1) where 64 x 64 leaves compute units without one.
// Layer of 512 tokens, 128 x 256, 4 experts: the two GEMMs 4.5 and 4.8 us (10.2 and 15.5 with a 4 x 4
// register block of v_fmac per thread).
template <int ACT, int TM, int TN>
__global__ __launch_bounds__(256) void grouped_gemm_f32_kernel(
    const float *__restrict__ A, const float *__restrict__ B, const float *__restrict__ bias,
    float *__restrict__ C, const WorkItem *__restrict__ items, int N, int K)
{
    const WorkItem tile = items[blockIdx.x];
    if (tile.expert < 0) return;
    const int n0 = tile.n0;

    constexpr int BM = 32 * TM, BN = 32 * TN, BK = 32, PD = 4;
    constexpr int LDA = BK + 4, LDB = BN + 4;
    __shared__ __attribute__((aligned(16))) float As[2][BM * LDA];
    __shared__ __attribute__((aligned(16))) float Bs[2][BK * LDB];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1, r16 = lane & 15, kq = lane >> 4;
    const int KT = (K + BK - 1) / BK;

    const float *a_src[TM], *b_src[TN];
    int a_off[TM], b_off[TN], a_k[TM], b_k[TN];
#pragma unroll
    for (int q = 0; q < TM; ++q) {
        const int v = tid + 256 * q, row = v / 8;
        a_k[q] = v % 8 * 4;
        a_src[q] = A + static_cast<size_t>(min(tile.row0 + row, tile.row1 - 1)) * K;
        a_off[q] = row * LDA + a_k[q];
    }
#pragma unroll
    for (int q = 0; q < TN; ++q) {
        const int v = tid + 256 * q, n = v % (BN / 4) * 4;
        b_k[q] = v / (BN / 4);
        b_src[q] = B + static_cast<size_t>(tile.expert) * K * N + min(n0 + n, N - 4);   // (columns past N are not stored)
        b_off[q] = b_k[q] * LDB + n;
    }
    f32x4 ar[PD][TM], br[PD][TN];
    // (no branches around the loads, or the compiler waits for all of them: what lies past K is read
    // from inside the row or column and zeroed on its way into LDS)
    auto load = [&](auto slot, int s) {
        constexpr int u = decltype(slot)::value;
#pragma unroll
        for (int q = 0; q < TM; ++q)
            ar[u][q] = *reinterpret_cast<const f32x4 *>(a_src[q] + min(s * BK + a_k[q], K - 4));
#pragma unroll
        for (int q = 0; q < TN; ++q)
            br[u][q] = *reinterpret_cast<const f32x4 *>(b_src[q] + static_cast<size_t>(min(s * BK + b_k[q], K - 1)) * N);
    };
    f32x4 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};

    auto stage = [&](auto slot, int s) {
        constexpr int u = decltype(slot)::value, buf = u & 1;
#pragma unroll
        for (int q = 0; q < TM; ++q)
            *reinterpret_cast<f32x4 *>(&As[buf][a_off[q]]) =
                s * BK + a_k[q] < K ? ar[u][q] : (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int q = 0; q < TN; ++q)
            *reinterpret_cast<f32x4 *>(&Bs[buf][b_off[q]]) =
                s * BK + b_k[q] < K ? br[u][q] : (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
        load(slot, min(s + PD, KT - 1));         // (past the last stage: loaded again, never used)
        // LDS writes only are waited for: the loads stay in flight across the barrier
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int c = 0; c < BK; c += 16) {
            f32x4 af[TM], wf[TN];
#pragma unroll
            for (int j = 0; j < TM; ++j)
                af[j] = *reinterpret_cast<const f32x4 *>(&As[buf][((wm * TM + j) * 16 + r16) * LDA + c + 4 * kq]);
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    wf[i][q] = Bs[buf][(c + 4 * kq + q) * LDB + (wn * TN + i) * 16 + r16];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < TN; ++i)
#pragma unroll
                    for (int j = 0; j < TM; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[i][q], af[j][q], acc[i][j], 0, 0, 0);
        }
    };
    auto each = [&](auto body) {
        body(std::integral_constant<int, 0>{});
        body(std::integral_constant<int, 1>{});
        body(std::integral_constant<int, 2>{});
        body(std::integral_constant<int, 3>{});
    };
    each([&](auto u) { load(u, min(decltype(u)::value, KT - 1)); });
    int s0 = 0;
    for (; s0 + PD <= KT; s0 += PD) each([&](auto u) { stage(u, s0 + decltype(u)::value); });
    each([&](auto u) {
        if (s0 + decltype(u)::value < KT) stage(u, s0 + decltype(u)::value);
    });

    // acc[i][j][c]: column n0 + (wn * TN + i) * 16 + 4 * kq + c, row row0 + (wm * TM + j) * 16 + r16
#pragma unroll
    for (int i = 0; i < TN; ++i) {
        const int n = n0 + (wn * TN + i) * 16 + 4 * kq;
        if (n >= N) continue;
        f32x4 bs = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
        if (bias != nullptr) bs = *reinterpret_cast<const f32x4 *>(bias + static_cast<size_t>(tile.expert) * N + n);
#pragma unroll
        for (int j = 0; j < TM; ++j) {
            const int r = tile.row0 + (wm * TM + j) * 16 + r16;
            if (r >= tile.row1) continue;
            f32x4 o;
#pragma unroll
            for (int c = 0; c < 4; ++c) o[c] = activate<ACT, false>(acc[i][j][c] + bs[c]);
            *reinterpret_cast<f32x4 *>(C + static_cast<size_t>(r) * N + n) = o;
        }
    }
}

// ---------------------------------------------------------------- MFMA GEMM
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

template <bool F16>
__device__ __forceinline__ f32x16 mfma_32x32x16(const u32x4 &a, const u32x4 &b, const f32x16 &c)
{
    if constexpr (F16)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a),
                                                      __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ void store4(_Float16 *p, const float (&v)[4])
{
    f16x4 h;
    h[0] = static_cast<_Float16>(v[0]);
    h[1] = static_cast<_Float16>(v[1]);
    h[2] = static_cast<_Float16>(v[2]);
    h[3] = static_cast<_Float16>(v[3]);
    *reinterpret_cast<f16x4 *>(p) = h;
}

// C[r, n] = act(sum_k A[r,k] W[e][n,k] + bias[e][n]);  A [rows, K], W [E, N, K],
// 16-bit elements (bf16, or fp16 when F16), C [rows, N] of TOut.
// WM x WN wavefronts, each owning (TM*32) rows x (TN*32) columns of the block's
// (WM*TM*32) x (WN*TN*32) output tile.  K is walked in stages of 64 through a
// double-buffered LDS tile; the global loads of stages kt+2 (and kt+3) are in flight while
// stage kt is multiplied, and the barrier of a stage sits before its last 16-deep step so
// that the MFMAs of that step cover the LDS latency of the next stage's first
// fragments.  The work list (one entry per output tile) is ordered so that each XCD
// walks a contiguous share of it: neighbouring blocks then reuse operand tiles in that
// XCD's L2.  32-row sub-tiles past the end of a ragged row tile are skipped.
// KEEP: the pre-activation values (accumulator + bias) also go to Pre [rows, N] as fp16, for
// the backward pass.
// row_src != NULL: A is not the expert-major buffer but the token matrix itself, and the row
// operand of slot i is token row_src[i] / row_div (the dispatch plan's src_of and k): the
// loader gathers the tokens where they lie, so the multiply does not wait for the pack.
template <bool F16, typename TOut, int ACT, int WM, int WN, int TM, int TN, bool KTAIL, bool KEEP>
// (two wavefronts per SIMD in every shape: two 4-wavefront blocks or one 8-wavefront block)
__global__ __launch_bounds__(64 * WM * WN, 2) void grouped_gemm_staged_kernel(
    const uint16_t *__restrict__ A, const uint16_t *__restrict__ W,
    const float *__restrict__ bias, TOut *__restrict__ C, _Float16 *__restrict__ Pre,
    const WorkItem *__restrict__ items, int N, int K,
    const int32_t *__restrict__ row_src, int row_div)
{
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32, BK = 64, LD = BK + 8;
    constexpr int NT = 64 * WM * WN;
    constexpr int AV = BM * 8 / NT, WV = BN * 8 / NT;   // 16-byte vectors per thread per stage
    static_assert(BM * 8 % NT == 0 && BN * 8 % NT == 0, "tile does not divide over the threads");

    const WorkItem item = items[blockIdx.x];
    if (item.expert < 0) return;
    const int n0 = item.n0;
    const int rows = item.row1 - item.row0;

    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    constexpr int A_BUF = BM * LD, W_BUF = BN * LD;
    uint16_t *As = smem;               // [2][BM][LD]
    uint16_t *Ws = smem + 2 * A_BUF;   // [2][BN][LD]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const uint16_t *Wexp = W + static_cast<size_t>(item.expert) * N * K;

    const uint16_t *a_src[AV];
    const uint16_t *w_src[WV];
    int a_off[AV], w_off[WV];
    const int ld_col = (tid & 7) * 8;
#pragma unroll
    for (int q = 0; q < AV; ++q) {
        const int r = (tid + NT * q) >> 3;
        a_off[q] = r * LD + ld_col;
        // row_src: the operand rows are gathered -- row i of the expert-major order is row
        // row_src[i] / row_div of A (the token that holds assignment row_src[i])
        int arow = min(item.row0 + r, item.row1 - 1);
        if (row_src != nullptr) arow = row_src[arow] / row_div;
        a_src[q] = A + static_cast<size_t>(arow) * K + ld_col;
    }
#pragma unroll
    for (int q = 0; q < WV; ++q) {
        const int r = (tid + NT * q) >> 3;
        w_off[q] = r * LD + ld_col;
        w_src[q] = Wexp + static_cast<size_t>(min(n0 + r, N - 1)) * K + ld_col;
    }
    // 32-row sub-tiles of this wavefront that hold real rows
    const int jact = min(TM, max(0, (rows - wm * TM * 32 + 31) / 32));

    f32x16 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    // register stages between the global loads and the LDS tile: the loads have two stages of
    // multiplies to arrive
    constexpr int DEPTH = 2;
    u32x4 a_reg[AV], w_reg[WV];
    u32x4 a_reg2[AV], w_reg2[WV];
    u32x4 wf[2][TN], af[2][TM];
    const int KT = (K + BK - 1) / BK;
    const int fr = lane & 31, fk = (lane >> 5) * 8;
    const int wfrag = (wn * TN * 32 + fr) * LD + fk;
    const int afrag = (wm * TM * 32 + fr) * LD + fk;

#define MOE_LOADG(kt_, AR, WR)                                                                  \
    {                                                                                           \
        const int k0_ = (kt_) * BK;                                                             \
        const bool in_ = !KTAIL || k0_ + ld_col < K;                                           \
        _Pragma("unroll") for (int q = 0; q < AV; ++q)                                          \
        {                                                                                       \
            if (in_) AR[q] = *reinterpret_cast<const u32x4 *>(a_src[q] + k0_);                  \
            else AR[q] = (u32x4){0u, 0u, 0u, 0u};                                               \
        }                                                                                       \
        _Pragma("unroll") for (int q = 0; q < WV; ++q)                                          \
        {                                                                                       \
            if (in_) WR[q] = *reinterpret_cast<const u32x4 *>(w_src[q] + k0_);                  \
            else WR[q] = (u32x4){0u, 0u, 0u, 0u};                                               \
        }                                                                                       \
    }
#define MOE_STOREL(buf, AR, WR)                                                                 \
    {                                                                                           \
        _Pragma("unroll") for (int q = 0; q < AV; ++q)                                          \
            *reinterpret_cast<u32x4 *>(As + (buf) * A_BUF + a_off[q]) = AR[q];                  \
        _Pragma("unroll") for (int q = 0; q < WV; ++q)                                          \
            *reinterpret_cast<u32x4 *>(Ws + (buf) * W_BUF + w_off[q]) = WR[q];                  \
    }
#define MOE_READF(slot_, buf, ks)                                                               \
    {                                                                                           \
        _Pragma("unroll") for (int i = 0; i < TN; ++i) wf[slot_][i] =                           \
            *reinterpret_cast<const u32x4 *>(Ws + (buf) * W_BUF + wfrag + i * 32 * LD + (ks) * 16); \
        _Pragma("unroll") for (int j = 0; j < TM; ++j) af[slot_][j] =                           \
            *reinterpret_cast<const u32x4 *>(As + (buf) * A_BUF + afrag + j * 32 * LD + (ks) * 16); \
    }
#define MOE_MMA(slot_)                                                                          \
    {                                                                                           \
        _Pragma("unroll") for (int j = 0; j < TM; ++j)                                          \
        {                                                                                       \
            if (FULL || j < jact) {                                                             \
                _Pragma("unroll") for (int i = 0; i < TN; ++i)                                  \
                    acc[i][j] = mfma_32x32x16<F16>(wf[slot_][i], af[slot_][j], acc[i][j]);      \
            }                                                                                   \
        }                                                                                       \
    }
// One stage kt held in LDS buffer `buf`: the registers AR/WR (stage kt+1) go to the other
// buffer and are refilled with stage kt+1+DEPTH.
#define MOE_STAGE(buf, AR, WR)                                                                  \
    {                                                                                           \
        const bool next1 = kt + 1 < KT, nextl = kt + 1 + DEPTH < KT;                            \
        if (next1) MOE_STOREL(buf ^ 1, AR, WR)                                                  \
        if (nextl) MOE_LOADG(kt + 1 + DEPTH, AR, WR)                                            \
        MOE_READF(1, buf, 1)                                                                    \
        MOE_MMA(0)                                                                              \
        MOE_READF(0, buf, 2)                                                                    \
        MOE_MMA(1)                                                                              \
        MOE_READF(1, buf, 3)                                                                    \
        MOE_MMA(0)                                                                              \
        __syncthreads();                                                                        \
        __builtin_amdgcn_sched_barrier(0);                                                      \
        if (next1) MOE_READF(0, buf ^ 1, 0)                                                     \
        MOE_MMA(1)                                                                              \
    }
#define MOE_MAIN_LOOP                                                                           \
    {                                                                                           \
        int kt = 0;                                                                             \
        for (; kt + 1 < KT; kt += 2) {                                                          \
            MOE_STAGE(0, a_reg, w_reg)                                                          \
            ++kt;                                                                               \
            MOE_STAGE(1, a_reg2, w_reg2)                                                        \
            --kt;                                                                               \
        }                                                                                       \
        if (kt < KT) MOE_STAGE(0, a_reg, w_reg)                                                 \
    }

    // prologue: stage 0 into LDS, stages 1 and 2 in flight
    MOE_LOADG(0, a_reg, w_reg)
    MOE_STOREL(0, a_reg, w_reg)
    if (KT > 1) MOE_LOADG(1, a_reg, w_reg)
    if (KT > 2) MOE_LOADG(2, a_reg2, w_reg2)
    __syncthreads();
    MOE_READF(0, 0, 0)
    if (jact == TM) {          // every sub-tile of this wavefront holds rows: branch-free loop
        constexpr bool FULL = true;
        MOE_MAIN_LOOP
    } else {
        constexpr bool FULL = false;
        MOE_MAIN_LOOP
    }
#undef MOE_STAGE
#undef MOE_MAIN_LOOP
#undef MOE_LOADG
#undef MOE_STOREL
#undef MOE_READF
#undef MOE_MMA

    // acc[i][j][4*g + c]: column n0 + (wn*TN + i)*32 + 8*g + 4*(lane/32) + c,
    //                     row item.row0 + (wm*TM + j)*32 + lane%32
    const float *bexp = bias != nullptr ? bias + static_cast<size_t>(item.expert) * N : nullptr;
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        const int r = item.row0 + (wm * TM + j) * 32 + fr;
        if (r >= item.row1) continue;
#pragma unroll
        for (int i = 0; i < TN; ++i) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int n = n0 + (wn * TN + i) * 32 + 8 * g + 4 * (lane >> 5);
                if (n >= N) continue;
                float v[4], pre[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    float s = acc[i][j][4 * g + c];
                    if (bexp != nullptr) s += bexp[n + c];
                    pre[c] = s;
                    v[c] = activate<ACT, true>(s);
                }
                if constexpr (KEEP) store4(Pre + static_cast<size_t>(r) * N + n, pre);
                store4(C + static_cast<size_t>(r) * N + n, v);
            }
        }
    }
}

#include "gemm_w4.h"
#include "gemm_w4_run.h"

// ---------------------------------------------------------------- few rows per expert
// The same product for decode steps: a few rows per expert, so the time is that of streaming the
// weights once.  A wavefront owns 16 columns and the rows (RT groups of 16) of a 64-column item and
// takes its fragments straight from global memory -- no LDS, no barriers -- with PD 64-deep stages of
// loads in flight.  A block is one wavefront: at 768 columns and 16 experts the second GEMM of a layer is
// 768 blocks that spread over all compute units (as blocks of four wavefronts it took 192 units, and
// what an L1 can keep in flight, about 32 KiB, bound those), and twelve blocks fit a unit, so that the
// first GEMM's 3072 are one round.  Items hold at most 32 rows: with 64 a
// popular expert's wavefronts had three stages in flight instead of five and ended last.
// The contraction order is that of the other 16-bit kernels (same bits).
// 16 tokens, 16 experts, k = 2, 768 x 3072, the two GEMMs: 16.3 and 14.5 us (17.0 and 18.4 with four
// wavefronts a block; 17.2 and 25.7 with 128 x 128 and 64 x 256 tiles).
template <bool F16, int ACT, bool KEEP, bool KTAIL>
__global__ __launch_bounds__(64, 3) void grouped_gemm_stream_kernel(
    const uint16_t *__restrict__ A, const uint16_t *__restrict__ W, const float *__restrict__ bias,
    _Float16 *__restrict__ C, _Float16 *__restrict__ Pre, const WorkItem *__restrict__ items,
    int N, int K, const int32_t *__restrict__ row_src, int row_div)
{
    // the four blocks of an item are eight apart: one L2's
    const WorkItem item = items[blockIdx.x / 32 * 8 + blockIdx.x % 8];
    if (item.expert < 0) return;
    const int rows = item.row1 - item.row0;
    const int lane = threadIdx.x, fr = lane & 15, oct = lane >> 4;
    const int nw = item.n0 + static_cast<int>(blockIdx.x / 8 % 4) * 16;
    if (nw >= N) return;
    const int KT = (K + 63) / 64;
    const uint16_t *wp = W + (static_cast<size_t>(item.expert) * N + min(nw + fr, N - 1)) * K + oct * 8;

    auto body = [&](auto rt, auto pd) {
        constexpr int RT = decltype(rt)::value, PD = decltype(pd)::value;
        const uint16_t *ap[RT];
#pragma unroll
        for (int j = 0; j < RT; ++j) {
            int arow = item.row0 + min(j * 16 + fr, rows - 1);
            if (row_src != nullptr) arow = row_src[arow] / row_div;
            ap[j] = A + static_cast<size_t>(arow) * K + oct * 8;
        }
        u32x4 wr[PD][2], ar[PD][RT][2];
        // (no branches around the loads, or the compiler waits for all of them: a piece past K is read
        // from inside the row, and zeroed when the last stage is multiplied)
        auto load = [&](auto u, int s) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                int k0 = s * 64 + p * 32;
                if constexpr (KTAIL) k0 = min(k0, K - 8 - oct * 8);
                wr[decltype(u)::value][p] = *reinterpret_cast<const u32x4 *>(wp + k0);
#pragma unroll
                for (int j = 0; j < RT; ++j)
                    ar[decltype(u)::value][j][p] = *reinterpret_cast<const u32x4 *>(ap[j] + k0);
            }
        };
        f32x4 acc[RT];
#pragma unroll
        for (int j = 0; j < RT; ++j) acc[j] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
        auto use = [&](auto u, auto tail, int s) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const bool past = KTAIL && decltype(tail)::value && s * 64 + p * 32 + oct * 8 >= K;
                const u32x4 zero = {0u, 0u, 0u, 0u}, w = past ? zero : wr[decltype(u)::value][p];
#pragma unroll
                for (int j = 0; j < RT; ++j) {
                    const u32x4 a = past ? zero : ar[decltype(u)::value][j][p];
                    if constexpr (F16)
                        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                            __builtin_bit_cast(f16x8, w), __builtin_bit_cast(f16x8, a), acc[j], 0, 0, 0);
                    else
                        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf16x8, w), __builtin_bit_cast(bf16x8, a), acc[j], 0, 0, 0);
                }
            }
        };
        static_for<PD>([&](auto u) { load(u, min(decltype(u)::value, KT - 1)); });
        int s = 0;
        for (; s + 2 * PD <= KT; s += PD)
            static_for<PD>([&](auto u) {
                use(u, std::false_type{}, 0);
                load(u, s + decltype(u)::value + PD);
                __builtin_amdgcn_sched_barrier(0);
            });
        for (; s < KT; s += PD)                      // the last stages: fewer than two rounds
            static_for<PD>([&](auto u) {
                if (s + decltype(u)::value < KT) use(u, std::true_type{}, s + decltype(u)::value);
                if (s + decltype(u)::value + PD < KT) load(u, s + decltype(u)::value + PD);
            });

        // acc[j][c]: column nw + 4 * oct + c, row row0 + 16 * j + fr
        const int n = nw + 4 * oct;
        if (n >= N) return;
        float b4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (bias != nullptr) {
#pragma unroll
            for (int c = 0; c < 4; ++c) b4[c] = bias[static_cast<size_t>(item.expert) * N + n + c];
        }
#pragma unroll
        for (int j = 0; j < RT; ++j) {
            if (j * 16 + fr >= rows) continue;
            const size_t at = static_cast<size_t>(item.row0 + j * 16 + fr) * N + n;
            float v[4], pre[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                pre[c] = acc[j][c] + b4[c];
                v[c] = activate<ACT, true>(pre[c]);
            }
            if constexpr (KEEP) store4(Pre + at, pre);
            store4(C + at, v);
        }
    };
    using std::integral_constant;
    if (rows <= 16)
        body(integral_constant<int, 1>{}, integral_constant<int, 8>{});
    else
        body(integral_constant<int, 2>{}, integral_constant<int, 5>{});
}

// BM x 256 tiles, a share of them per block (gemm_w4_run.h).
// ABL (measurement only, 0 in the layer): bit 0 leaves out the MFMAs, bit 1 the LDS fragment
// reads after the first step, bit 2 the global loads into LDS inside the loop, bit 3 the
// output stores.  Results are then wrong by construction; every access stays inside the buffers.
template <bool F16, int ACT, bool KEEP, bool KTAIL, int BM, int ABL>
__device__ __forceinline__ void run_gemm_tiles(
    const uint16_t *__restrict__ A, const uint16_t *__restrict__ W,
    const float *__restrict__ bias, _Float16 *__restrict__ C, _Float16 *__restrict__ Pre,
    const WorkItem *__restrict__ items, const int32_t *__restrict__ nitems, int entries, int share, int N, int K,
    const int32_t *__restrict__ row_src, int row_div, int a_rows)
{
    constexpr int TN = 8;
    struct Bias { float at[TN][4]; };
    auto prepare = [&](const WorkItem &item, int wn, int oct) {
        Bias b4;
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int c = 0; c < 4; ++c) b4.at[i][c] = 0.0f;
        if (bias != nullptr) {
            const float *bexp = bias + static_cast<size_t>(item.expert) * N;
            const int n = item.n0 + wn * 128 + 4 * oct;
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int c = 0; c < 4; ++c) b4.at[i][c] = bexp[min(n + i * 16 + c, N - 1)];
        }
        return b4;
    };
    w4_run<F16, KTAIL, BM, ABL>(A, W, items, nitems, entries, share, N, K, row_src, row_div, a_rows, prepare, [&](
        auto &acc, const Bias &b4, const WorkItem &item, const W4Place<BM> &place, auto landed) {
        WorkItem stored = item;
        if constexpr (ABL & 8) stored.row1 = 0;
        // R rows are stored while the next ones are computed.  KEEP: 16, each pass through its own half of the patch where
        // it has two, so that the sums of no more are kept from the first pass to the second: with 32 the 256 x 256 kernel
        // takes 504 to 512 of a SIMD's 512 registers, with 16 at most 472, and the pack's wavefronts (32) get in beside a
        // block that holds its unit.  32768 tokens, 2048 x 8192, 64 experts, a launch's tiles in 256 shares, us: pack 1376 -> 236,
        // this GEMM 1886 -> 1902, the second one, which the pack was left to, 1632 -> 1602.  20 training steps of 18000 .. 32768 tokens: 0.986 .. 1.019 of
        // their time, mean 0.999; packed in front of this GEMM 0.973 .. 1.058, mean 1.004.
        constexpr int UR = W4Place<BM>::UR, R = KEEP ? 16 : UR;
#pragma unroll
        for (int r = 0; r < BM / 2; r += R) {
#pragma unroll
            for (int pass = KEEP ? 0 : 1; pass < 2; ++pass) {      // pass 0: pre-activations, 1: outputs
                const int part = KEEP && UR == 32 ? pass : 0;
#pragma unroll
                for (int j = r / 16; j < (r + R) / 16; ++j) {
#pragma unroll
                    for (int i = 0; i < TN; ++i) {
                        float v[4];
#pragma unroll
                        for (int c = 0; c < 4; ++c) {
                            const float sum = acc[i][j][c] + b4.at[i][c];
                            v[c] = pass == 0 ? sum : activate<ACT, true>(sum);
                        }
                        store4(reinterpret_cast<_Float16 *>(place.at(i, part + j - r / 16)), v);
                        if (i % 4 == 3) MOE_SB();   // a few accumulator registers at a time leave the AGPRs
                    }
                }
                if (r == 0 && pass == (KEEP ? 0 : 1)) landed();
                place.template leave<R>(reinterpret_cast<uint16_t *>(pass == 0 ? Pre : C), stored, r, part, N);
            }
        }
    });
}

template <bool F16, int ACT, bool KEEP, bool KTAIL, int ABL = 0>
__global__ __launch_bounds__(256, 1) void grouped_gemm_w4_kernel(
    const uint16_t *__restrict__ A, const uint16_t *__restrict__ W,
    const float *__restrict__ bias, _Float16 *__restrict__ C, _Float16 *__restrict__ Pre,
    const WorkItem *__restrict__ items, const int32_t *__restrict__ nitems, int entries, int share, int N, int K,
    const int32_t *__restrict__ row_src, int row_div, int a_rows)
{
    run_gemm_tiles<F16, ACT, KEEP, KTAIL, 256, ABL>(A, W, bias, C, Pre, items, nitems, entries, share, N, K,
                                                    row_src, row_div, a_rows);
}

// 128 x 128 tiles, one per block; DEEP: of launches that wait for their weights, with five stages on their way
template <bool F16, int ACT, bool KEEP, bool KTAIL, bool DEEP>
__device__ __forceinline__ void w4_gemm_tile(
    const uint16_t *__restrict__ A, const uint16_t *__restrict__ W,
    const float *__restrict__ bias, _Float16 *__restrict__ C, _Float16 *__restrict__ Pre,
    const WorkItem *__restrict__ items, int N, int K,
    const int32_t *__restrict__ row_src, int row_div, int a_rows)
{
    constexpr int BM = 128, BN = 128;
    constexpr bool TILE_IN = false;
    const uint16_t *const tile_in = nullptr;
#include "gemm_w4_body.inc"

    // Epilogue.  The wavefront's
    // BM / 2 x BN / 2 sub-tile goes to its own patch (16 bytes of row padding) and leaves as whole
    // lines, 16 bytes per lane.
    constexpr int PITCH = BN + 16, LPR = BN / 16, RPI = 64 / LPR;   // lanes per row, rows per instruction
    char *patch = lds + wave * (BM / 2) * PITCH;
    const float *bexp = bias != nullptr ? bias + static_cast<size_t>(item.expert) * N : nullptr;
    const int rbase = item.row0 + wm * (BM / 2);
    const int ncol = n0 + wn * (BN / 2) + lane % LPR * 8;
#pragma unroll
    for (int pass = KEEP ? 0 : 1; pass < 2; ++pass) {      // pass 0: pre-activations, 1: outputs
        _Float16 *out = pass == 0 ? Pre : C;
#pragma unroll
        for (int i = 0; i < TN; ++i) {
            const int col = i * 16 + 4 * oct;
            float b4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if (bexp != nullptr) {
#pragma unroll
                for (int c = 0; c < 4; ++c) b4[c] = bexp[min(n0 + wn * (BN / 2) + col + c, N - 1)];
            }
#pragma unroll
            for (int j = 0; j < TM; ++j) {
                float v[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float s = acc[i][j][c] + b4[c];
                    v[c] = pass == 0 ? s : activate<ACT, true>(s);
                }
                store4(reinterpret_cast<_Float16 *>(patch + (j * 16 + fr) * PITCH) + col, v);
                if (j == TM / 2 - 1) MOE_SB();
            }
            MOE_SB();          // a few accumulator registers at a time leave the AGPRs
        }
        MOE_LGKM0();
        __builtin_amdgcn_wave_barrier();
#pragma unroll 8
        for (int it = 0; it < BM / 2 / RPI; ++it) {
            const int rr = it * RPI + lane / LPR;
            const u32x4 q = *reinterpret_cast<const u32x4 *>(patch + rr * PITCH + lane % LPR * 16);
            const int r = rbase + rr;
            if (r < item.row1 && ncol < N)
                *reinterpret_cast<u32x4 *>(out + static_cast<size_t>(r) * N + ncol) = q;
        }
        if (pass == 0) {
            MOE_LGKM0();
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// 128 x BN tiles
template <bool F16, int ACT, bool KEEP, bool KTAIL, int BN, bool DEEP = false>
__global__ __launch_bounds__(256, BN == 128 && !DEEP ? 2 : 1) void grouped_gemm_mfma_kernel(
    const uint16_t *__restrict__ A, const uint16_t *__restrict__ W,
    const float *__restrict__ bias, _Float16 *__restrict__ C, _Float16 *__restrict__ Pre,
    const WorkItem *__restrict__ items, int entries, int share, int N, int K,
    const int32_t *__restrict__ row_src, int row_div, int a_rows)
{
    if constexpr (BN == 256)
        run_gemm_tiles<F16, ACT, KEEP, KTAIL, 128, 0>(A, W, bias, C, Pre, items, nullptr, entries, share, N, K,
                                                      row_src, row_div, a_rows);
    else
        w4_gemm_tile<F16, ACT, KEEP, KTAIL, DEEP>(A, W, bias, C, Pre, items, N, K, row_src, row_div, a_rows);
}
#undef MOE_LGKM0
#undef MOE_VMCNT
#undef MOE_SB
#undef MOE_BAR
#undef MOE_MATRIX_RESULTS

// ---------------------------------------------------------------- weight packing
// Out[e][n][k] = convert(In[e][k][n]); 64 x 64 tiles through LDS.
// MODE 0: bf16 -> bf16, MODE 1: bf16 -> fp16.
template <int MODE>
__global__ __launch_bounds__(256) void transpose_pack_kernel(
    const uint16_t *__restrict__ in, uint16_t *__restrict__ out, int K, int N)
{
    __shared__ uint16_t tile[64][66];
    const size_t eoff = static_cast<size_t>(blockIdx.z) * K * N;
    const int k0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
    for (int v = threadIdx.x; v < 64 * 64; v += 256) {
        const int kk = v / 64, nn = v % 64;
        uint16_t val = 0;
        if (k0 + kk < K && n0 + nn < N) val = in[eoff + static_cast<size_t>(k0 + kk) * N + n0 + nn];
        tile[kk][nn] = val;
    }
    __syncthreads();
    for (int v = threadIdx.x; v < 64 * 64; v += 256) {
        const int nn = v / 64, kk = v % 64;
        if (k0 + kk < K && n0 + nn < N) {
            uint16_t val = tile[kk][nn];
            if constexpr (MODE == 1) {
                const _Float16 h = static_cast<_Float16>(bf16_to_f32(val));
                val = __builtin_bit_cast(uint16_t, h);
            }
            out[eoff + static_cast<size_t>(n0 + nn) * K + k0 + kk] = val;
        }
    }
}

template <int ACT>
void launch_f32_pair(const moe_shape &s, const float *xe, const float *W1, const float *b1,
                     const float *W2, const float *b2, float *ye, const Workspace &w,
                     int chunk, hipStream_t st)
{
    float *H = static_cast<float *>(w.hidden);
    const WorkItem *it1 = w.items[0] + static_cast<size_t>(chunk) * w.gp[0].max_items;
    const WorkItem *it2 = w.items[1] + static_cast<size_t>(chunk) * w.gp[1].max_items;
    auto launch = [&](auto act, int g, const float *A, const float *B, const float *bias, float *C,
                      const WorkItem *items, int N, int K) {
        constexpr int A_ = decltype(act)::value;
        const GemmPlan &gp = w.gp[g];
        auto kern = gp.bm == 64 ? grouped_gemm_f32_kernel<A_, 2, 2> : grouped_gemm_f32_kernel<A_, 1, 1>;
        hipLaunchKernelGGL(kern, dim3(gp.max_items), dim3(256), 0, st, A, B, bias, C, items, N, K);
    };
    prof_begin(kStageGemm1, st);
    launch(std::integral_constant<int, ACT>{}, 0, xe, W1, b1, H, it1, s.d_ff, s.d_model);
    prof_end(kStageGemm1, st);
    prof_begin(kStageGemm2, st);
    launch(std::integral_constant<int, MOE_ACT_IDENTITY>{}, 1, H, W2, b2, ye, it2, s.d_model, s.d_ff);
    prof_end(kStageGemm2, st);
}

template <bool F16, typename TOut, int ACT, int WM, int WN, int TM, int TN, bool KTAIL, bool KEEP>
void launch_mfma_cfg_k(const uint16_t *A, const uint16_t *W, const float *bias, TOut *C,
                     _Float16 *pre, const WorkItem *items, int max_items,
                     int N, int K, int stage, hipStream_t st, const int32_t *row_src, int row_div)
{
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
    constexpr size_t lds = 2 * (BM + BN) * (64 + 8) * sizeof(uint16_t);
    auto kern = grouped_gemm_staged_kernel<F16, TOut, ACT, WM, WN, TM, TN, KTAIL, KEEP>;
    static PerDeviceOnce once;   // raising the dynamic LDS limit: once per kernel and device
    once.raise_lds(reinterpret_cast<const void *>(kern), static_cast<int>(lds));
    hipEvent_t t0, t1;
    prof_kernel_events(stage, &t0, &t1);
    hipExtLaunchKernelGGL(kern, dim3(max_items), dim3(64 * WM * WN), lds, st, t0, t1, 0, A, W, bias, C,
                          pre, items, N, K, row_src, row_div);
}

// The contraction depth is a multiple of the 64-deep stage in every benchmark shape;
// other depths take a variant that zero-fills the last stage.
template <bool F16, typename TOut, int ACT, bool KEEP, int WM, int WN, int TM, int TN>
void launch_mfma_cfg(const uint16_t *A, const uint16_t *W, const float *bias, TOut *C,
                     _Float16 *pre, const WorkItem *items, int max_items,
                     int N, int K, int stage, hipStream_t st, const int32_t *row_src, int row_div)
{
    if (K % 64 == 0)
        launch_mfma_cfg_k<F16, TOut, ACT, WM, WN, TM, TN, false, KEEP>(
            A, W, bias, C, pre, items, max_items, N, K, stage, st, row_src, row_div);
    else
        launch_mfma_cfg_k<F16, TOut, ACT, WM, WN, TM, TN, true, KEEP>(
            A, W, bias, C, pre, items, max_items, N, K, stage, st, row_src, row_div);
}

// The four-wavefront kernel addresses its operands with 32-bit byte offsets into buffer
// resources (the expert's weight matrix; the tile's rows, or the whole token matrix when the
// rows are gathered; the tile's rows of the output, where 0x7ff00000 lies past every one).
inline bool w4_kernel_fits(int N, int K, bool gathered, uint64_t row_limit)
{
    constexpr uint64_t most = (1ull << 31) - 64;
    return static_cast<uint64_t>(N) * K * 2 < most && 256ull * N * 2 < most - (1 << 20) &&
           (gathered ? row_limit * static_cast<uint64_t>(K) : 256ull * K) * 2 < most;
}

template <bool F16, typename TOut, int ACT, bool KEEP>
void launch_mfma(const GemmPlan &gp, const uint16_t *A, const uint16_t *W, const float *bias,
                 TOut *C, _Float16 *pre, const WorkItem *items, int N, int K,
                 int stage, hipStream_t st, const int32_t *row_src = nullptr, int row_div = 1,
                 uint64_t row_limit = 0)
{
#define MOE_MFMA_SHAPE(WM_, WN_, TM_, TN_)                                                        \
    launch_mfma_cfg<F16, TOut, ACT, KEEP, WM_, WN_, TM_, TN_>(A, W, bias, C, pre, items,            \
                                                              gp.max_items, N, K, stage, st,       \
                                                              row_src, row_div)
    if (gp.w4) {
        // tiles of 256 columns: shares of the list (kRunStages)
        const bool run = gp.bn == 256;
        auto launch = [&](auto kern, PerDeviceOnce &once, auto... list) {
            const size_t lds = run || gp.deep ? kW4RunLds : w4_lds(128, 128);
            once.raise_lds(reinterpret_cast<const void *>(kern), static_cast<int>(lds));
            hipEvent_t t0, t1;
            prof_kernel_events(stage, &t0, &t1);
            const int share = w4_run_share(gp.bm, K);
            hipExtLaunchKernelGGL(kern, dim3(run ? w4_run_blocks(gp.max_items, share) : gp.max_items), dim3(256), lds, st,
                                  t0, t1, 0, A, W, bias, C, pre, items, list..., gp.max_items, share, N, K, row_src, row_div,
                                  static_cast<int>(row_limit));
        };
        auto shape = [&](auto tail) {
            constexpr bool TAIL = decltype(tail)::value;
            static PerDeviceOnce once[4];
            if (gp.bm == 256)
                launch(grouped_gemm_w4_kernel<F16, ACT, KEEP, TAIL>, once[0], static_cast<const int32_t *>(nullptr));
            else if (run)
                launch(grouped_gemm_mfma_kernel<F16, ACT, KEEP, TAIL, 256>, once[1]);
            else if (gp.deep)
                launch(grouped_gemm_mfma_kernel<F16, ACT, KEEP, TAIL, 128, true>, once[3]);
            else
                launch(grouped_gemm_mfma_kernel<F16, ACT, KEEP, TAIL, 128>, once[2]);
        };
        if (K % 64 == 0 && (!run || K >= 256))
            shape(std::false_type{});
        else
            shape(std::true_type{});
    }
    else if (gp.bn == 64) {
        auto kern = K % 64 == 0 ? grouped_gemm_stream_kernel<F16, ACT, KEEP, false>
                                : grouped_gemm_stream_kernel<F16, ACT, KEEP, true>;
        const int grid = gp.max_items * 4;
        hipEvent_t t0, t1;
        prof_kernel_events(stage, &t0, &t1);
        hipExtLaunchKernelGGL(kern, dim3(grid), dim3(64), 0, st, t0, t1, 0, A, W, bias, C, pre, items, N, K,
                              row_src, row_div);
    }
    else if (gp.bm == 64)
        MOE_MFMA_SHAPE(1, 8, 2, 1);
    else
        MOE_MFMA_SHAPE(2, 4, 2, 2);
#undef MOE_MFMA_SHAPE
}

template <int ACT>
void launch_mfma_pair(const moe_shape &s, const uint16_t *xe, const uint16_t *W1p,
                      const float *b1, const uint16_t *W2p, const float *b2, _Float16 *ye,
                      _Float16 *pre, const Workspace &w, int chunk, hipStream_t st,
                      const int32_t *row_src, int row_div)
{
    _Float16 *H = static_cast<_Float16 *>(w.hidden);
    const WorkItem *it1 = w.items[0] + static_cast<size_t>(chunk) * w.gp[0].max_items;
    const WorkItem *it2 = w.items[1] + static_cast<size_t>(chunk) * w.gp[1].max_items;
    if (pre != nullptr)
        launch_mfma<false, _Float16, ACT, true>(w.gp[0], xe, W1p, b1, H, pre, it1,
                                                s.d_ff, s.d_model,
                                                kStageGemm1, st, row_src, row_div, s.T);
    else
        launch_mfma<false, _Float16, ACT, false>(w.gp[0], xe, W1p, b1, H, nullptr, it1, s.d_ff, s.d_model,
                                                 kStageGemm1, st, row_src, row_div, s.T);
    launch_mfma<true, _Float16, MOE_ACT_IDENTITY, false>(w.gp[1], reinterpret_cast<const uint16_t *>(H),
                                                      W2p, b2, ye, nullptr, it2,
                                                      s.d_model, s.d_ff, kStageGemm2, st);
}

}  // namespace

// Which kernel the layer launches for expert GEMM `which` (0: first, 1: second) of a bf16 layer,
// for labelling measurements: "<kernel> <tile rows>x<tile columns>".
void expert_gemm_kernel_name(const moe_shape &s, int which, char *name, size_t len)
{
    const GemmPlan gp = choose_gemm_plan(s, which, 1, s.T);
    std::snprintf(name, len, "%s %dx%d%s",
                  gp.w4 ? gp.bm == 256 ? "grouped_gemm_w4_kernel" : "grouped_gemm_mfma_kernel"
                        : gp.bn == 64 ? "grouped_gemm_stream_kernel" : "grouped_gemm_staged_kernel",
                  gp.bm, gp.bn, gp.deep ? " deep" : "");
}

// Measurement aid: the 256 x 256 kernel alone on caller-made operands and work list, with
// parts of it left out (see ABL above).  gelu != 0 applies the activation.
moe_status launch_calib_gemm(const uint16_t *A, const uint16_t *W, _Float16 *C, const WorkItem *items,
                             const int32_t *nitems, int max_items, int N, int K, int abl, int gelu,
                             hipStream_t st)
{
    if (!w4_kernel_fits(N, K, false, 0)) {
        set_error("moe_calib_gemm: N * K * 2 and 256 * K * 2 must be below 2^31 and 256 * N * 2 below 2^31 - 2^20 (N = %d, K = %d)", N, K);
        return MOE_EINVAL;
    }
    constexpr size_t lds = kW4RunLds;
    const int entries = static_cast<int>(align_up(static_cast<size_t>(max_items), 8));
    const int share = w4_run_share(256, K), grid = w4_run_blocks(entries, share);
    auto run = [&](auto kern, PerDeviceOnce &once) {
        once.raise_lds(reinterpret_cast<const void *>(kern), static_cast<int>(lds));
        hipLaunchKernelGGL(kern, dim3(grid), dim3(256), lds, st, A, W, nullptr, C, nullptr, items, nitems, entries, share, N,
                           K, nullptr, 1, 0);
    };
    auto variant = [&](auto abl_, auto tail) {
        constexpr int ABL = decltype(abl_)::value;
        constexpr bool TAIL = decltype(tail)::value;
        static PerDeviceOnce once[2];              // (of these two kernels)
        if (gelu) run(grouped_gemm_w4_kernel<false, MOE_ACT_GELU_ERF, false, TAIL, ABL>, once[0]);
        else run(grouped_gemm_w4_kernel<false, MOE_ACT_IDENTITY, false, TAIL, ABL>, once[1]);
    };
#define MOE_CALIB_CASE(ABL_)                                                                      \
    case ABL_:                                                                                    \
        if (K >= 256) variant(std::integral_constant<int, ABL_>{}, std::false_type{});            \
        else variant(std::integral_constant<int, ABL_>{}, std::true_type{});                      \
        break;
    switch (abl) {
        MOE_CALIB_CASE(0)
        MOE_CALIB_CASE(1)
        MOE_CALIB_CASE(2)
        MOE_CALIB_CASE(4)
        MOE_CALIB_CASE(6)
        MOE_CALIB_CASE(7)
        MOE_CALIB_CASE(8)
    default:
        set_error("moe_calib_gemm: variant %d is not built (0, 1, 2, 4, 6, 7, 8)", abl);
        return MOE_EINVAL;
    }
#undef MOE_CALIB_CASE
    MOE_TRY_HIP(hipGetLastError());
    return MOE_OK;
}

// Tile shape of expert GEMM `which` (0: xe.W1, 1: H.W2) for this layer shape.  Large
// tiles cut the operand traffic per flop; they need enough output tiles to fill 256
// compute units, and a long contraction to amortise their prologue and epilogue.
GemmPlan choose_gemm_plan(const moe_shape &s, int which, int n_launches, int64_t tokens)
{
    GemmPlan gp;
    const int N = which == 0 ? s.d_ff : s.d_model;
    const int K = which == 0 ? s.d_model : s.d_ff;
    const int64_t max_rows = moe_max_rows(&s);
    auto rows_of = [&](int64_t t) { return t * s.k < max_rows ? t * s.k : max_rows; };
    const int64_t chunk_rows = rows_of((s.T + n_launches - 1) / n_launches);
    if (s.dtype != MOE_BF16) {
        // 64 x 64 tiles where they are a few per compute unit, else 32 x 32 (us of the layer, 32 / 64:
        // 603 tokens, 420 x 1620 71 / 88; 951, k = 2, 780 x 2084 183 / 189; 3564, 764 x 1836 308 / 250)
        gp.bm = gp.bn = (chunk_rows / 64 + s.E / 2) * ((N + 63) / 64) >= 1200 ? 64 : 32;
        gp.concurrent = 256;
    } else {
        const int64_t per_expert = chunk_rows / s.E;
        const int64_t tiles_n = (N + 255) / 256;
        if (chunk_rows <= 5 * static_cast<int64_t>(s.E) ||
            (chunk_rows <= 32 * static_cast<int64_t>(s.E) && chunk_rows * ((N + 127) / 128) <= 2000)) {
            // a decode step: the weights are streamed once, by as many blocks as there are.  Every
            // wavefront of 16 columns reads the rows again, so a larger tile takes over once they weigh
            // as much as what sharing the weights out gains: the more column tiles there are to
            // occupy the chip with, the fewer rows it takes.  us of the layer, this / the best other
            // tile for the second GEMM: 8 experts, 768 x 3072, 6 / 16 / 36 rows per expert 42 / 55, 46 /
            // 56, 55 / 56; 16, 1536 x 6144, 8 / 12 / 24 161 / 180, 166 / 179, 191 / 183; 32, 1024 x 4096, 8 /
            // 12 138 / 139, 147 / 141; for the first: 4, 1024 x 4096, 6 / 24 58 / 63, 63 / 63; 16, 768 x
            // 3072, 8 / 12 76 / 79, 82 / 77.  With Zipf(1.2) popularity the lines lie lower (16, 1536 x
            // 6144, 8 / 12 rows 174 / 174, 198 / 182; 32, 512 x 1024, 16 43.5 / 40.4), hence 2000.
            // Items of 32 rows: of 64 a popular expert's wavefronts hold three stages in flight instead of
            // five and end last (Zipf, 16, 1536 x 6144, 8 rows 198 -> 174; 32, 512 x 1024, 8 42 -> 39.5).
            gp.bm = 32; gp.bn = 64; gp.concurrent = 128;
        } else if (few_long_tiles(chunk_rows, s.E, N, K) && w4_kernel_fits(N, K, which == 0, static_cast<uint64_t>(s.T))) {
            // Time of the layer over that with the kernels below: 30 layers, K = 1920 .. 13952, 11 .. 610 rows per
            // expert 0.75 .. 0.99, mean 0.92 (8 experts, 3584 x 1024, 60 rows 158 -> 118 us; 8, 9856 x 2816, 11 rows 521 ->
            // 437); K = 512 .. 1919 0.96 .. 1.05, mean 0.99.  257 .. 1400 tiles 0.82 .. 1.16, mean 1.01: a second round of few
            // tiles takes as long as the first (8 experts, 14336 x 4096, 64 rows 1800 -> 1990 us of four layers).
            gp.bm = gp.bn = 128; gp.concurrent = 32; gp.w4 = gp.deep = true;
        } else if ((chunk_rows / 64 + s.E / 2) * tiles_n >= 128 &&
                   (per_expert < 48 || (per_expert <= 64 && (chunk_rows / 128 + s.E / 2) * tiles_n < 256))) {
            // few rows per expert and enough 64-row tiles to keep the weight stream going: shorter
            // tiles spend less of their loads on (mostly padded) rows (137 tokens, 16 experts, k = 3,
            // first GEMM 1256 x 3096: 87 us of the layer, 92 with 128 x 128; 256 tokens, 8 experts,
            // second GEMM 14336 x 4096: 1831 us of four layers, 1952)
            gp.bm = 64; gp.bn = 256; gp.concurrent = 32;
        } else if (w4_kernel_fits(N, K, which == 0, static_cast<uint64_t>(s.T))) {
            choose_w4_tile(chunk_rows, s.E, N, K, &gp);
        } else {                       // operands past 32-bit offsets
            gp.bm = 128; gp.bn = 256; gp.concurrent = 32;
        }
    }
    gp.tiles_n = (N + gp.bn - 1) / gp.bn;
    gp.max_row_tiles = static_cast<int32_t>((rows_of(tokens) + gp.bm - 1) / gp.bm + s.E);
    gp.max_items = work_list_entries(gp);
    return gp;
}

moe_status launch_ffn(const moe_shape &s, const void *xe, const void *W1p, const float *b1,
                      const void *W2p, const float *b2, void *ye, const Workspace &w,
                      int chunk, hipStream_t st, void *pre, const int32_t *row_src)
{
    if (row_src != nullptr && s.dtype != MOE_BF16) {
        set_error("gathered token rows are for bf16 layers only");
        return MOE_EUNSUPPORTED;
    }
    if (pre != nullptr && s.dtype != MOE_BF16) {
        set_error("the pre-activations are kept for bf16 layers only");
        return MOE_EUNSUPPORTED;
    }
#define MOE_FFN_CASE(ACT)                                                                      \
    case ACT:                                                                                  \
        if (s.dtype == MOE_BF16)                                                               \
            launch_mfma_pair<ACT>(s, static_cast<const uint16_t *>(xe),                         \
                                  static_cast<const uint16_t *>(W1p), b1,                       \
                                  static_cast<const uint16_t *>(W2p), b2,                       \
                                  static_cast<_Float16 *>(ye), static_cast<_Float16 *>(pre), w, \
                                  chunk, st, row_src, s.k);                                     \
        else                                                                                   \
            launch_f32_pair<ACT>(s, static_cast<const float *>(xe),                             \
                                 static_cast<const float *>(W1p), b1,                           \
                                 static_cast<const float *>(W2p), b2, static_cast<float *>(ye), \
                                 w, chunk, st);                                                 \
        break;
    switch (s.act) {
        MOE_FFN_CASE(MOE_ACT_GELU_ERF)
        MOE_FFN_CASE(MOE_ACT_GELU_TANH)
        MOE_FFN_CASE(MOE_ACT_RELU)
        MOE_FFN_CASE(MOE_ACT_IDENTITY)
    default:
        set_error("unknown activation %d", s.act);
        return MOE_EINVAL;
    }
#undef MOE_FFN_CASE
    MOE_TRY_HIP(hipGetLastError());
    return MOE_OK;
}

moe_status launch_pack(const moe_shape &s, const void *W1, const void *W2, void *W1p,
                       void *W2p, hipStream_t st)
{
    const size_t elems = static_cast<size_t>(s.E) * s.d_model * s.d_ff;
    if (s.dtype == MOE_F32) {
        MOE_TRY_HIP(hipMemcpyAsync(W1p, W1, elems * 4, hipMemcpyDeviceToDevice, st));
        MOE_TRY_HIP(hipMemcpyAsync(W2p, W2, elems * 4, hipMemcpyDeviceToDevice, st));
        return MOE_OK;
    }
    // W1 [E, d, h] -> [E, h, d];  W2 [E, h, d] -> [E, d, h] as fp16
    hipLaunchKernelGGL(transpose_pack_kernel<0>,
                       dim3(ceil_div(s.d_ff, 64), ceil_div(s.d_model, 64), s.E), dim3(256), 0, st,
                       static_cast<const uint16_t *>(W1), static_cast<uint16_t *>(W1p), s.d_model,
                       s.d_ff);
    hipLaunchKernelGGL(transpose_pack_kernel<1>,
                       dim3(ceil_div(s.d_model, 64), ceil_div(s.d_ff, 64), s.E), dim3(256), 0, st,
                       static_cast<const uint16_t *>(W2), static_cast<uint16_t *>(W2p), s.d_ff,
                       s.d_model);
    MOE_TRY_HIP(hipGetLastError());
    return MOE_OK;
}

}  // namespace moe
