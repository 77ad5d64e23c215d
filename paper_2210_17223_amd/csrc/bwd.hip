// Backward pass of the MoE layer (chain rule of the forward of paper Sec. 2.1; the paper
// trains this layer and schedules its backward pass in Sec. 2.2 and Sec. 4).
//
//   combine_bwd      dye[slot] = g dy[t] (bf16), dgate = <ye[slot], dy[t]>
//   gemm (rows)      P = xe W1 (fp16) and Hb = act(P) (bf16) -- only when the forward did not
//                    keep P and its hidden activations
//   gemm (rows)      dP = (dye W2^T) * act'(P)                        (bf16)
//   gemm (rows)      dxe = dP W1^T                                    (fp32)
//   gemm (wgrad)     dW2[e] = act(P)^T dye, dW1[e] = xe^T dP          (fp32), operands row-major
//                    as they are: the fragments come out of LDS through transposing reads
//   gate_bwd         logits (from the packed gate matrix), softmax, dz,
//                    dx = sum of the token's dxe rows + dz Wg^T
//   dwg              dWg = x^T dz (partial sums over token ranges, then a fixed-order sum)
//
// The row-grouped GEMMs run on the forward's four-wavefront kernels (gemm_w4.h) and its kind of
// work list; a weight-gradient GEMM contracts over one expert's rows.
#include "activation.h"
#include "common.h"
#include "moe_train.h"

#include <algorithm>
#include <cstdio>

#include <hip/hip_ext.h>

namespace moe {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;

#include "gemm_w4.h"

constexpr int kBM = 128, kBN = 256, kBK = 64, kLD = kBK + 8;
constexpr size_t kGemmLds = 2 * (kBM + kBN) * kLD * sizeof(uint16_t);

template <int ACT>
__device__ __forceinline__ float act_value(float v)
{
    if constexpr (ACT == MOE_ACT_GELU_ERF)
        return gelu_erf_fast(v);
    else if constexpr (ACT == MOE_ACT_GELU_TANH)
        return v * half_one_plus_tanh(v);
    else if constexpr (ACT == MOE_ACT_RELU)
        return fmaxf(v, 0.0f);
    else
        return v;
}

template <int ACT>
__device__ __forceinline__ float act_derivative(float v)
{
    if constexpr (ACT == MOE_ACT_GELU_ERF) {
        return gelu_erf_derivative_fast(v);
    } else if constexpr (ACT == MOE_ACT_GELU_TANH) {
        // s = (1 + tanh u) / 2:  s + v s' with s' = 2 s (1 - s) u'
        const float c = 0.7978845608028654f, a = 0.044715f, s = half_one_plus_tanh(v);
        return s + 2.0f * v * s * (1.0f - s) * c * (1.0f + 3.0f * a * v * v);
    } else if constexpr (ACT == MOE_ACT_RELU) {
        return v > 0.0f ? 1.0f : 0.0f;
    } else {
        return 1.0f;
    }
}

__device__ __forceinline__ void store_bf16x4(uint16_t *p, const float (&v)[4])
{
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    u32x2 o;                       // (the packed conversion: the bits of f32_to_bf16)
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        bf16x2 b;
        b[0] = static_cast<__bf16>(v[2 * c]);
        b[1] = static_cast<__bf16>(v[2 * c + 1]);
        o[c] = __builtin_bit_cast(uint32_t, b);
    }
    *reinterpret_cast<u32x2 *>(p) = o;
}

// ---------------------------------------------------------------- combine backward
// One wavefront per token.
__global__ __launch_bounds__(256) void combine_bwd_kernel(
    const float *__restrict__ dy, const _Float16 *__restrict__ ye, const int32_t *__restrict__ slot_of,
    const float *__restrict__ gate, uint16_t *__restrict__ dye, float *__restrict__ dgate, int t0,
    int T, int d, int k, int max_rows)
{
    // tokens [t0, T)
    const int lane = lane_id();
    const int t = t0 + blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (t >= T) return;
    const float *dyrow = dy + static_cast<size_t>(t) * d;
    for (int j = 0; j < k; ++j) {
        const int slot = slot_of[static_cast<size_t>(t) * k + j];
        if (slot < 0 || slot >= max_rows) {
            if (lane == 0) dgate[static_cast<size_t>(t) * k + j] = 0.0f;
            continue;
        }
        const float g = gate[static_cast<size_t>(t) * k + j];
        const _Float16 *yerow = ye + static_cast<size_t>(slot) * d;
        uint16_t *out = dye + static_cast<size_t>(slot) * d;
        float dot = 0.0f;
        for (int c = lane * 4; c < d; c += kWave * 4) {
            const float4 a = *reinterpret_cast<const float4 *>(dyrow + c);
            typedef __attribute__((ext_vector_type(4))) _Float16 half4;
            const half4 b = *reinterpret_cast<const half4 *>(yerow + c);
            dot = __builtin_fmaf(a.x, static_cast<float>(b[0]), dot);
            dot = __builtin_fmaf(a.y, static_cast<float>(b[1]), dot);
            dot = __builtin_fmaf(a.z, static_cast<float>(b[2]), dot);
            dot = __builtin_fmaf(a.w, static_cast<float>(b[3]), dot);
            const float v[4] = {g * a.x, g * a.y, g * a.z, g * a.w};
            store_bf16x4(out + c, v);
        }
#pragma unroll
        for (int m = kWave / 2; m > 0; m >>= 1) dot += __shfl_xor(dot, m);
        if (lane == 0) dgate[static_cast<size_t>(t) * k + j] = dot;
    }
}

// ---------------------------------------------------------------- GEMM
// (For operands that the four-wavefront kernels' 32-bit offsets do not reach.)
// C[r, n] = sum_k A[r, k] W[e][n, k] for the rows of one work item.
// EPI 0: fp32 store.  EPI 1: P = acc as fp16 into Pbuf and act(acc) as bf16 into C.
// EPI 2: acc * act'(Pbuf) as bf16 into C.
template <int EPI, int ACT, bool KTAIL>
__global__ __launch_bounds__(512, 2) void bwd_gemm_kernel(
    const uint16_t *__restrict__ A, const uint16_t *__restrict__ W, void *__restrict__ Cout,
    _Float16 *__restrict__ Pbuf, const WorkItem *__restrict__ items, int N, int K)
{
    constexpr int WM = 2, TM = 2, TN = 2, NT = 512;        // 2 x 4 wavefronts of 64 x 64
    constexpr int AV = kBM * 8 / NT, WV = kBN * 8 / NT;
    int expert, row0, row1, n0;
    {
        const WorkItem item = items[blockIdx.x];
        if (item.expert < 0) return;
        expert = item.expert; row0 = item.row0; row1 = item.row1; n0 = item.n0;
    }
    const int KT = (K + kBK - 1) / kBK;
    const size_t w_base = static_cast<size_t>(expert) * N * K;
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    constexpr int A_BUF = kBM * kLD, W_BUF = kBN * kLD;
    uint16_t *As = smem;
    uint16_t *Ws = smem + 2 * A_BUF;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int fr = lane & 31, fk = (lane >> 5) * 8;

    f32x16 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    if (KT > 0) {
        const uint16_t *a_src[AV];
        const uint16_t *w_src[WV];
        int a_off[AV], w_off[WV];
        const int ld_col = (tid & 7) * 8;
#pragma unroll
        for (int q = 0; q < AV; ++q) {
            const int r = (tid + NT * q) >> 3;
            a_off[q] = r * kLD + ld_col;
            a_src[q] = A + static_cast<size_t>(min(row0 + r, row1 - 1)) * K + ld_col;
        }
#pragma unroll
        for (int q = 0; q < WV; ++q) {
            const int r = (tid + NT * q) >> 3;
            w_off[q] = r * kLD + ld_col;
            w_src[q] = W + w_base + static_cast<size_t>(min(n0 + r, N - 1)) * K + ld_col;
        }
        u32x4 a_reg[AV], w_reg[WV], a_reg2[AV], w_reg2[WV];   // two register stages of prefetch
        u32x4 wf[2][TN], af[2][TM];
        const int wfrag = (wn * TN * 32 + fr) * kLD + fk;
        const int afrag = (wm * TM * 32 + fr) * kLD + fk;
#define BWD_LOADG(kt_, AR, WR)                                                                  \
    {                                                                                           \
        const int k0_ = (kt_) * kBK;                                                            \
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
#define BWD_STOREL(buf, AR, WR)                                                                 \
    {                                                                                           \
        _Pragma("unroll") for (int q = 0; q < AV; ++q)                                          \
            *reinterpret_cast<u32x4 *>(As + (buf) * A_BUF + a_off[q]) = AR[q];                  \
        _Pragma("unroll") for (int q = 0; q < WV; ++q)                                          \
            *reinterpret_cast<u32x4 *>(Ws + (buf) * W_BUF + w_off[q]) = WR[q];                  \
    }
#define BWD_READF(slot_, buf, ks)                                                               \
    {                                                                                           \
        _Pragma("unroll") for (int i = 0; i < TN; ++i) wf[slot_][i] =                           \
            *reinterpret_cast<const u32x4 *>(Ws + (buf) * W_BUF + wfrag + i * 32 * kLD + (ks) * 16); \
        _Pragma("unroll") for (int j = 0; j < TM; ++j) af[slot_][j] =                           \
            *reinterpret_cast<const u32x4 *>(As + (buf) * A_BUF + afrag + j * 32 * kLD + (ks) * 16); \
    }
#define BWD_MMA(slot_)                                                                          \
    {                                                                                           \
        _Pragma("unroll") for (int j = 0; j < TM; ++j)                                          \
            _Pragma("unroll") for (int i = 0; i < TN; ++i)                                      \
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(                            \
                    __builtin_bit_cast(bf16x8, wf[slot_][i]),                                   \
                    __builtin_bit_cast(bf16x8, af[slot_][j]), acc[i][j], 0, 0, 0);              \
    }
// stage kt in LDS buffer `buf`: AR/WR (stage kt+1) go to the other buffer and are refilled
// with stage kt+3
#define BWD_STAGE(buf, AR, WR)                                                                  \
    {                                                                                           \
        const bool next1 = kt + 1 < KT, next3 = kt + 3 < KT;                                    \
        if (next1) BWD_STOREL(buf ^ 1, AR, WR)                                                  \
        if (next3) BWD_LOADG(kt + 3, AR, WR)                                                    \
        BWD_READF(1, buf, 1)                                                                    \
        BWD_MMA(0)                                                                              \
        BWD_READF(0, buf, 2)                                                                    \
        BWD_MMA(1)                                                                              \
        BWD_READF(1, buf, 3)                                                                    \
        BWD_MMA(0)                                                                              \
        __syncthreads();                                                                        \
        __builtin_amdgcn_sched_barrier(0);                                                      \
        if (next1) BWD_READF(0, buf ^ 1, 0)                                                     \
        BWD_MMA(1)                                                                              \
    }
        BWD_LOADG(0, a_reg, w_reg)
        BWD_STOREL(0, a_reg, w_reg)
        if (KT > 1) BWD_LOADG(1, a_reg, w_reg)
        if (KT > 2) BWD_LOADG(2, a_reg2, w_reg2)
        __syncthreads();
        BWD_READF(0, 0, 0)
        int kt = 0;
        for (; kt + 1 < KT; kt += 2) {
            BWD_STAGE(0, a_reg, w_reg)
            ++kt;
            BWD_STAGE(1, a_reg2, w_reg2)
            --kt;
        }
        if (kt < KT) BWD_STAGE(0, a_reg, w_reg)
#undef BWD_STAGE
#undef BWD_LOADG
#undef BWD_STOREL
#undef BWD_READF
#undef BWD_MMA
    }

    // acc[i][j][4*g + c]: column n0 + (wn*TN + i)*32 + 8*g + 4*(lane/32) + c,
    //                     row row0 + (wm*TM + j)*32 + lane%32
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        const int r = row0 + (wm * TM + j) * 32 + fr;
        if (r >= row1) continue;
#pragma unroll
        for (int i = 0; i < TN; ++i) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int n = n0 + (wn * TN + i) * 32 + 8 * g + 4 * (lane >> 5);
                if (n >= N) continue;
                const size_t at = static_cast<size_t>(r) * N + n;
                float v[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = acc[i][j][4 * g + c];
                if constexpr (EPI == 0) {
                    *reinterpret_cast<float4 *>(static_cast<float *>(Cout) + at) =
                        make_float4(v[0], v[1], v[2], v[3]);
                } else if constexpr (EPI == 1) {
                    f16x4 p;
                    float a[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        p[c] = static_cast<_Float16>(v[c]);
                        a[c] = act_value<ACT>(v[c]);
                    }
                    *reinterpret_cast<f16x4 *>(Pbuf + at) = p;
                    store_bf16x4(static_cast<uint16_t *>(Cout) + at, a);
                } else {
                    const f16x4 p = *reinterpret_cast<const f16x4 *>(Pbuf + at);
                    float a[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) a[c] = v[c] * act_derivative<ACT>(static_cast<float>(p[c]));
                    store_bf16x4(static_cast<uint16_t *>(Cout) + at, a);
                }
            }
        }
    }
}

// ---------------------------------------------------------------- GEMM, four wavefronts
// The same three products on the forward's four-wavefront layout (gemm_w4.h).  The tile leaves through LDS as
// whole lines (16-bit outputs) or straight from the registers (fp32); for EPI 2 the tile of
// pre-activations is in LDS when the loop ends.
template <int EPI, int ACT, bool KTAIL, int BM, int BN, bool DEEP = false>
__global__ __launch_bounds__(256, BM + BN == 256 && !DEEP ? 2 : 1) void bwd_gemm_w4_kernel(
    const uint16_t *__restrict__ A, const uint16_t *__restrict__ W, void *__restrict__ Cout,
    _Float16 *__restrict__ Pbuf, const WorkItem *__restrict__ items, int N, int K)
{
    constexpr bool F16 = false;
    const int32_t *const row_src = nullptr;      // packed rows
    constexpr int row_div = 1, a_rows = 0;
    constexpr bool TILE_IN = EPI == 2;
    const uint16_t *const tile_in = reinterpret_cast<const uint16_t *>(Pbuf);
#include "gemm_w4_body.inc"

    const int rbase = item.row0 + wm * (BM / 2);
    if constexpr (EPI == 0) {
        float *out = static_cast<float *>(Cout);
#pragma unroll
        for (int i = 0; i < TN; ++i) {
            const int n = n0 + wn * (BN / 2) + i * 16 + 4 * oct;
#pragma unroll
            for (int j = 0; j < TM; ++j) {
                const int r = rbase + j * 16 + fr;
                if (r < item.row1 && n < N)
                    *reinterpret_cast<float4 *>(out + static_cast<size_t>(r) * N + n) =
                        make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
                if (j == TM / 2 - 1) MOE_SB();
            }
            MOE_SB();          // a few accumulator registers at a time leave the AGPRs
        }
    } else if constexpr (EPI == 2) {
        // The pre-activations are turned into dP in their places, 32 rows at a time, which leave while the next
        // are computed.
        constexpr int LPR = BN / 16, RPI = 64 / LPR;
        const int unit[4] = {RING5 ? ua : uw, RING5 ? uw : uw1, ua1, uw1};
        const int ncol = n0 + wn * (BN / 2) + lane % LPR * 8;
        uint16_t *out = static_cast<uint16_t *>(Cout);
        MOE_VMCNT(TILE_UNITS == 4 ? 2 * TILE_LOADS : 0);
        f16x4 p[2][TN];
        auto place = [&](int i, int j) {
            const int row = (j & 1) * 16 + fr;
            return lds + unit[j >> 1] + wave * (W_UNIT / 4) + row * BN + (((2 * i + (oct >> 1)) ^ tile_key(row)) << 4) +
                   (oct & 1) * 8;
        };
#pragma unroll
        for (int i = 0; i < TN; ++i) p[0][i] = *reinterpret_cast<const f16x4 *>(place(i, 0));
#pragma unroll
        for (int u = 0; u < TILE_UNITS; ++u) {
            char *const patch = lds + unit[u] + wave * (W_UNIT / 4);
#pragma unroll
            for (int j = 2 * u; j < 2 * u + 2; ++j) {
                if (j + 1 < TM) {                // (ahead of the writes, which the compiler would keep in front)
#pragma unroll
                    for (int i = 0; i < TN; ++i) p[(j + 1) & 1][i] = *reinterpret_cast<const f16x4 *>(place(i, j + 1));
                }
#pragma unroll
                for (int i = 0; i < TN; ++i) {
                    float a[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        a[c] = acc[i][j][c] * act_derivative<ACT>(static_cast<float>(p[j & 1][i][c]));
                    store_bf16x4(reinterpret_cast<uint16_t *>(place(i, j)), a);
                    if (i % 4 == 3) MOE_SB();   // a few accumulator registers at a time leave the AGPRs
                }
            }
            // (the last units, before any store is: nothing younger than they)
            if (u == 0 && TILE_UNITS == 4) MOE_VMCNT(0);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int it = 0; it < 32 / RPI; ++it) {
                const int rr = it * RPI + lane / LPR, r = rbase + u * 32 + rr;
                const u32x4 q = *reinterpret_cast<const u32x4 *>(patch + rr * BN + ((lane % LPR ^ tile_key(rr)) << 4));
                if (r < item.row1 && ncol < N)
                    *reinterpret_cast<u32x4 *>(out + static_cast<size_t>(r) * N + ncol) = q;
            }
            MOE_SB();
        }
    } else {
        // the wavefront's BM / 2 x BN / 2 patch of 16-bit values; lanes per row, rows per instruction
        constexpr int PITCH = BN + 16, LPR = BN / 16, RPI = 64 / LPR;
        char *patch = lds + wave * (BM / 2) * PITCH;
        const int ncol = n0 + wn * (BN / 2) + lane % LPR * 8;
#pragma unroll
        for (int pass = 0; pass < 2; ++pass) {     // pass 0: the pre-activations
#pragma unroll
            for (int i = 0; i < TN; ++i) {
#pragma unroll
                for (int j = 0; j < TM; ++j) {
                    char *at = patch + (j * 16 + fr) * PITCH + (i * 16 + 4 * oct) * 2;
                    if (pass == 0) {
                        f16x4 p;
#pragma unroll
                        for (int c = 0; c < 4; ++c) p[c] = static_cast<_Float16>(acc[i][j][c]);
                        *reinterpret_cast<f16x4 *>(at) = p;
                    } else {
                        float a[4];
#pragma unroll
                        for (int c = 0; c < 4; ++c) a[c] = act_value<ACT>(acc[i][j][c]);
                        store_bf16x4(reinterpret_cast<uint16_t *>(at), a);
                    }
                    if (j == TM / 2 - 1) MOE_SB();
                }
                MOE_SB();
            }
            MOE_LGKM0();
            __builtin_amdgcn_wave_barrier();
            // whole row pieces from the patch to a [rows, N] matrix of 16-bit values
            uint16_t *dst = pass == 0 ? reinterpret_cast<uint16_t *>(Pbuf) : static_cast<uint16_t *>(Cout);
#pragma unroll 8
            for (int it = 0; it < BM / 2 / RPI; ++it) {
                const int rr = it * RPI + lane / LPR;
                const u32x4 q = *reinterpret_cast<const u32x4 *>(patch + rr * PITCH + lane % LPR * 16);
                const int r = rbase + rr;
                if (r < item.row1 && ncol < N)
                    *reinterpret_cast<u32x4 *>(dst + static_cast<size_t>(r) * N + ncol) = q;
            }
            if (pass == 0) {
                MOE_LGKM0();
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
}

// ---------------------------------------------------------------- weight gradient, row-major operands
// C[e][m, n] = sum over the rows r of expert e of A[r, m] B[r, n]: both operands are stored
// with the contraction index (the row) as the SLOW one.  The tiles go to LDS as they are --
// 64 rows x 128 columns, 16-byte vectors -- and the MFMA fragments (eight consecutive rows for
// one column per lane) come out of LDS through gfx950's transposing 64-bit read, which hands
// each lane of a 16-lane group four consecutive ROWS of one column: lane i of the group points
// at row i / 4, columns 4 (i % 4) .. + 3, and receives rows 0 .. 3 of column i.  The 64-byte
// pieces of a row are XOR-swizzled with the row number so that the four rows a group reads
// fall into different banks.  128 x 128 output tile, four wavefronts, the row-grouped GEMM's
// software pipeline; rows beyond the expert's last one are zeroed in the last stage only.
typedef __attribute__((ext_vector_type(4))) short s16x4;

__device__ __forceinline__ u32x2 lds_read_tr16(const uint16_t *p)
{
    const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) s16x4 *)(p));
    return __builtin_bit_cast(u32x2, v);
}

// AF16: A holds fp16 values (the forward's hidden activations); they are rounded to bf16 on
// their way into LDS (two conversions to fp32 and one packed conversion per pair).
template <int HALF>
__device__ __forceinline__ float f16_half_to_f32(uint32_t w)
{
    typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
    return static_cast<float>(__builtin_bit_cast(f16x2, w)[HALF]);
}
// (written out: between the matrix instructions the compiler converts the two one by one and merges them)
__device__ __forceinline__ uint32_t f32x2_to_bf16x2(float lo, float hi)
{
    uint32_t w = 0;
#if defined(__HIP_DEVICE_COMPILE__)
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(w) : "v"(lo), "v"(hi));
#endif
    return w;
}
__device__ __forceinline__ uint32_t f16x2_to_bf16x2(uint32_t w)
{
    return f32x2_to_bf16x2(f16_half_to_f32<0>(w), f16_half_to_f32<1>(w));
}

template <bool AF16>
__global__ __launch_bounds__(256, 2) void wgrad_gemm_kernel(
    const uint16_t *__restrict__ A, const uint16_t *__restrict__ B, float *__restrict__ C,
    const int32_t *__restrict__ offsets, int E, int M, int N, int tiles_m, int tiles_n)
{
    constexpr int WM = 2, TM = 2, TN = 2, NT = 256;     // 2 x 2 wavefronts of 64 x 64
    constexpr int kTile = 128, kRowB = kTile * 2;        // tile columns, bytes per LDS row
    constexpr int kBuf = kBK * kTile;                    // elements per LDS buffer
    constexpr int V = kBK * (kTile / 8) / NT;            // 16-byte vectors per thread, stage, operand
    int expert, m0, n0;
    {
        const int total = E * tiles_m * tiles_n;
        const int per_xcd = (total + 7) / 8;
        const int slot = blockIdx.x / 8;
        const int idx = (blockIdx.x % 8) * per_xcd + slot;
        if (slot >= per_xcd || idx >= total) return;
        expert = idx / (tiles_m * tiles_n);
        const int rem = idx % (tiles_m * tiles_n);
        m0 = (rem / tiles_n) * kTile;
        n0 = (rem % tiles_n) * kTile;
    }
    const int r0 = offsets[expert], r1 = offsets[expert + 1];
    const int KT = (r1 - r0 + kBK - 1) / kBK;
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    uint16_t *As = smem;                 // [2][kBK][kTile], swizzled
    uint16_t *Bs = smem + 2 * kBuf;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;

    f32x16 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    if (KT > 0) {
        // staging: vector v = tid + 256 q is row v / 16, columns 8 (v % 16) .. + 7 of the tile
        int st_row[V], st_off[V];
        size_t a_col[V], b_col[V];
        const uint16_t *a_ptr[V], *b_ptr[V];
#pragma unroll
        for (int q = 0; q < V; ++q) {
            const int v = tid + NT * q;
            const int k = v >> 4, c16 = v & 15;
            st_row[q] = k;
            st_off[q] = (k * kRowB + (((c16 >> 2) ^ (k & 3)) << 6) + ((c16 & 3) << 4)) >> 1;   // elements
            a_col[q] = static_cast<size_t>(min(m0 + c16 * 8, M - 8));
            b_col[q] = static_cast<size_t>(min(n0 + c16 * 8, N - 8));
            a_ptr[q] = A + static_cast<size_t>(r0 + k) * M + a_col[q];
            b_ptr[q] = B + static_cast<size_t>(r0 + k) * N + b_col[q];
        }
        const size_t a_step = static_cast<size_t>(kBK) * M, b_step = static_cast<size_t>(kBK) * N;
        u32x4 a_reg[V], b_reg[V], a_reg2[V], b_reg2[V];
        u32x4 bf[2][TN], af[2][TM];
        // fragment addresses: lane = 16 g + i reads row 8 (g / 2) + i / 4 (+ 4 for the upper
        // half) of the 16-row step, columns 16 (g % 2) + 4 (i % 4) .. + 3 of the 32-column sub-tile
        const int fi = lane & 15, fg = lane >> 4;
        const int frow = 8 * (fg >> 1) + (fi >> 2);
        const int fcol = 16 * (fg & 1) + 4 * (fi & 3);
// Stages are loaded in ascending order: the pointers walk 64 rows per call; only a stage that
// reaches past the expert's last row (the last one) clamps its rows and zeroes the surplus.
#define WG_LOADG(kt_, AR, BR)                                                                   \
    {                                                                                           \
        const int rbase_ = r0 + (kt_) * kBK;                                                    \
        if (rbase_ + kBK <= r1) {                                                               \
            _Pragma("unroll") for (int q = 0; q < V; ++q)                                       \
            {                                                                                   \
                AR[q] = *reinterpret_cast<const u32x4 *>(a_ptr[q]);                             \
                BR[q] = *reinterpret_cast<const u32x4 *>(b_ptr[q]);                             \
                a_ptr[q] += a_step;                                                             \
                b_ptr[q] += b_step;                                                             \
            }                                                                                   \
        } else {                                                                                \
            _Pragma("unroll") for (int q = 0; q < V; ++q)                                       \
            {                                                                                   \
                const int row_ = rbase_ + st_row[q];                                            \
                const size_t at_ = static_cast<size_t>(min(row_, r1 - 1));                      \
                AR[q] = *reinterpret_cast<const u32x4 *>(A + at_ * M + a_col[q]);               \
                BR[q] = *reinterpret_cast<const u32x4 *>(B + at_ * N + b_col[q]);               \
                if (row_ >= r1) {                                                               \
                    AR[q] = (u32x4){0u, 0u, 0u, 0u};                                            \
                    BR[q] = (u32x4){0u, 0u, 0u, 0u};                                            \
                }                                                                               \
            }                                                                                   \
        }                                                                                       \
    }
#define WG_STOREL(buf, AR, BR)                                                                  \
    {                                                                                           \
        _Pragma("unroll") for (int q = 0; q < V; ++q)                                           \
        {                                                                                       \
            u32x4 av_ = AR[q];                                                                  \
            if constexpr (AF16)                                                                 \
                av_ = (u32x4){f16x2_to_bf16x2(av_[0]), f16x2_to_bf16x2(av_[1]),                 \
                              f16x2_to_bf16x2(av_[2]), f16x2_to_bf16x2(av_[3])};                \
            *reinterpret_cast<u32x4 *>(As + (buf) * kBuf + st_off[q]) = av_;                    \
            *reinterpret_cast<u32x4 *>(Bs + (buf) * kBuf + st_off[q]) = BR[q];                  \
        }                                                                                       \
    }
// eight consecutive rows of one column per lane: two transposing reads, four rows each
#define WG_FRAG(dst, base, cb, ks)                                                              \
    {                                                                                           \
        const int col_ = (cb) + fcol;                                                           \
        const int k_ = (ks) * 16 + frow;                                                        \
        const int lo_ = (k_ * kRowB + (((col_ >> 5) ^ (k_ & 3)) << 6) + ((col_ & 31) << 1)) >> 1; \
        const u32x2 l_ = lds_read_tr16((base) + lo_);                                           \
        const u32x2 h_ = lds_read_tr16((base) + lo_ + 4 * kTile);                               \
        dst = (u32x4){l_[0], l_[1], h_[0], h_[1]};                                              \
    }
#define WG_READF(slot_, buf, ks)                                                                \
    {                                                                                           \
        _Pragma("unroll") for (int i = 0; i < TN; ++i)                                          \
            WG_FRAG(bf[slot_][i], Bs + (buf) * kBuf, (wn * TN + i) * 32, ks)                    \
        _Pragma("unroll") for (int j = 0; j < TM; ++j)                                          \
            WG_FRAG(af[slot_][j], As + (buf) * kBuf, (wm * TM + j) * 32, ks)                    \
    }
#define WG_MMA(slot_)                                                                           \
    {                                                                                           \
        _Pragma("unroll") for (int j = 0; j < TM; ++j)                                          \
            _Pragma("unroll") for (int i = 0; i < TN; ++i)                                      \
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(                            \
                    __builtin_bit_cast(bf16x8, bf[slot_][i]),                                   \
                    __builtin_bit_cast(bf16x8, af[slot_][j]), acc[i][j], 0, 0, 0);              \
    }
#define WG_STAGE(buf, AR, BR)                                                                   \
    {                                                                                           \
        const bool next1 = kt + 1 < KT, next3 = kt + 3 < KT;                                    \
        if (next1) WG_STOREL(buf ^ 1, AR, BR)                                                   \
        if (next3) WG_LOADG(kt + 3, AR, BR)                                                     \
        WG_READF(1, buf, 1)                                                                     \
        WG_MMA(0)                                                                               \
        WG_READF(0, buf, 2)                                                                     \
        WG_MMA(1)                                                                               \
        WG_READF(1, buf, 3)                                                                     \
        WG_MMA(0)                                                                               \
        __syncthreads();                                                                        \
        __builtin_amdgcn_sched_barrier(0);                                                      \
        if (next1) WG_READF(0, buf ^ 1, 0)                                                      \
        WG_MMA(1)                                                                               \
    }
        WG_LOADG(0, a_reg, b_reg)
        WG_STOREL(0, a_reg, b_reg)
        if (KT > 1) WG_LOADG(1, a_reg, b_reg)
        if (KT > 2) WG_LOADG(2, a_reg2, b_reg2)
        __syncthreads();
        WG_READF(0, 0, 0)
        int kt = 0;
        for (; kt + 1 < KT; kt += 2) {
            WG_STAGE(0, a_reg, b_reg)
            ++kt;
            WG_STAGE(1, a_reg2, b_reg2)
            --kt;
        }
        if (kt < KT) WG_STAGE(0, a_reg, b_reg)
#undef WG_STAGE
#undef WG_LOADG
#undef WG_STOREL
#undef WG_FRAG
#undef WG_READF
#undef WG_MMA
    }

    // acc[i][j][4*g + c]: column n0 + (wn*TN + i)*32 + 8*g + 4*(lane/32) + c,
    //                     row m0 + (wm*TM + j)*32 + lane%32
    float *Ce = C + static_cast<size_t>(expert) * M * N;
    const int fr = lane & 31;
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        const int m = m0 + (wm * TM + j) * 32 + fr;
        if (m >= M) continue;
#pragma unroll
        for (int i = 0; i < TN; ++i) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int n = n0 + (wn * TN + i) * 32 + 8 * g + 4 * (lane >> 5);
                if (n >= N) continue;
                *reinterpret_cast<float4 *>(Ce + static_cast<size_t>(m) * N + n) =
                    make_float4(acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2],
                                acc[i][j][4 * g + 3]);
            }
        }
    }
}

// ---------------------------------------------------------------- weight gradient, 256 x 256 tiles
// The same product on the four-wavefront layout of gemm_w4.h (operands straight into LDS, accumulators in AGPRs,
// every memory instruction between two matrix instructions), for layers whose weight gradients have enough
// 256 x 256 tiles.  A tile is few steps of 32 rows deep, so a block works through a share of the tiles
// and its loads run on across them: LDS is a ring of five steps of 32 KiB (32 rows x 256 columns of both
// operands), and while step s is multiplied the fragments of s + 1 are read, s + 2 .. s + 4 are on their way and
// s + 5 is requested into the step's own place, whether it belongs to this tile or the next.  A finished tile
// leaves through the place of its last step while the next one's first steps are there already.
// The fragments of the 16 x 16 x 32 instruction (eight rows of one column per lane) are two transposing
// LDS reads each.  The 64-byte pieces of a row are XOR-swizzled with the row's low two bits and its 32-byte
// halves with bit 3, so that the four rows of a 16-lane group, and two groups eight rows apart, fall into
// different banks.  The operands' buffer resources end with the expert's last row: rows past it -- and whole steps
// past the last one -- read as zeros, without clamping or tail code.
// AF16: A holds fp16 values, rounded to bf16 between the LDS read and the multiply, beside the column before.
//
// us of dW2 / dW1, one block per tile before / a share of the tiles per block: 63622 rows, 2048 x 8192, 64 experts
// 2742 / 2363 -> 2422 / 2137; 8192 rows, 768 x 3072, 16 experts 88 / 77 -> 75 / 68.  Of dW1's 2130 the matrix
// instructions with their LDS reads and barriers take 1275 by themselves, the loads beside them 320 more, the stores
// 350 (a unit's wavefronts wait until the 256 KiB of a tile are accepted; alone the 4.3 GB take 690, 6.2 TB/s),
// the way through LDS 110.  No wait for a load costs anything: not waiting at all is no faster.  The loads,
// one behind each column of instructions: 3 % / 2 % less than two at a time, 5 % / 4 % less than among the LDS
// reads.  The stores are two rows of 512 bytes per instruction: straight from the accumulators, 16 rows of 64
// bytes, past the caches the 4.3 GB alone take 1430 us, through them the operands are pushed out (dW1 2380).
// Blocks that start one after the other over the length of a tile, so that they do not store all at once: 2 %
// less for dW1, nothing for dW2.  Tiles in squares of 4 x 4: dW1 2455 -> 2325 with one block per tile.
// All of that with the tiles in 256 shares; in shares that give the unit back (kRunStages) 2417 / 2213 where those take 2379 / 2106.
template <bool AF16>
__global__ __launch_bounds__(256, 1) void wgrad_w4_kernel(
    const uint16_t *__restrict__ A, const uint16_t *__restrict__ B, float *__restrict__ C,
    const int32_t *__restrict__ offsets, int E, int M, int N, int tiles_m, int tiles_n, int share)
{
    constexpr int TM = 8, TN = 8, HALF = 16384, STEP = 2 * HALF, RING = 5;
    constexpr int kRow = 512;                     // bytes of a 256-column LDS row
    const int total = E * tiles_m * tiles_n;
    constexpr int stride = kRunUnits / 8;
    const int per_xcd = (total + 7) / 8, slot = blockIdx.x / 8, xcd = blockIdx.x % 8;
    int tile = xcd * per_xcd + slot / stride * stride * share + slot % stride;
    const int end = min(min(total, (xcd + 1) * per_xcd), tile + share * stride);
    if (tile >= end) return;
    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    char *const lds = reinterpret_cast<char *>(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int fr = lane & 15, oct = lane >> 4;
    const int first_row = offsets[min(lane, E)], end_row = offsets[min(lane + 1, E)];

    struct Tile {
        int expert, m0, n0, row0, rows;
        __device__ __forceinline__ int steps() const { return max((rows + 63) / 64 * 2, 2); }
    };
    auto tile_at = [&](int idx) {
        Tile t;
        t.expert = __builtin_amdgcn_readfirstlane(idx / (tiles_m * tiles_n));
        // squares of 4 x 4 tiles, along n inside a band of four: the 32 tiles an XCD has in flight share 12
        // panels of the operands whatever the matrix's shape (row by row, 33 of a wide one's)
        int rem = idx - t.expert * (tiles_m * tiles_n);
        const int band = rem / (4 * tiles_n), high = min(4, tiles_m - 4 * band);
        rem -= band * 4 * tiles_n;
        const int square = rem / (4 * high), wide = min(4, tiles_n - 4 * square);
        rem -= square * 4 * high;
        t.m0 = __builtin_amdgcn_readfirstlane((4 * band + rem / wide) * 256);
        t.n0 = __builtin_amdgcn_readfirstlane((4 * square + rem % wide) * 256);
        t.row0 = __builtin_amdgcn_readlane(first_row, t.expert);
        t.rows = __builtin_amdgcn_readlane(end_row, t.expert) - t.row0;
        return t;
    };

    // Loads: of the tile `load_tile`, `load_steps` more steps, from a_at / b_at (the tile's first column of the
    // step's first row); a_left / b_left bytes to the end of the expert's last row.
    int load_tile = tile, load_steps, a_left, b_left;
    const uint16_t *a_at, *b_at;
    auto open = [&]() {
        if (load_tile < end) {
            const Tile t = tile_at(load_tile);
            a_at = A + static_cast<size_t>(t.row0) * M + t.m0;
            b_at = B + static_cast<size_t>(t.row0) * N + t.n0;
            a_left = t.rows > 0 ? (t.rows * M - t.m0) * 2 : 0;
            b_left = t.rows > 0 ? (t.rows * N - t.n0) * 2 : 0;
            load_steps = t.steps();
        } else {                                  // (behind the last tile: zeros, never used)
            a_left = b_left = 0;
            load_steps = 0x7fffffff;
        }
    };
    // load q of this wavefront's four of an operand's step: rows wave * 8 + 2 q and + 1, 32 pieces of 16
    // bytes each; lane l lands at row l / 32, place l % 32
    int a_src[4], b_src[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int row = wave * 8 + q * 2 + (lane >> 5), place = lane & 31;
        const int piece = (place ^ ((row & 3) << 2)) ^ (((row >> 3) & 1) << 1);
        a_src[q] = (row * M + piece * 8) * 2;
        b_src[q] = (row * N + piece * 8) * 2;
    }
    const uint32_t dest = lds_address(lds) + wave * 4096;
    __amdgpu_buffer_rsrc_t rsa, rsb;
    // (the range check that turns rows past the expert's end into zeros sees the per-lane offset only)
    auto aim = [&]() {
        rsa = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(a_at), 0, static_cast<unsigned>(max(a_left, 0)), 0x00020000);
        rsb = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(b_at), 0, static_cast<unsigned>(max(b_left, 0)), 0x00020000);
    };
    auto load = [&](auto vc, int at) {            // load v (0 .. 7) of a step into the ring at `at`
        constexpr int v = decltype(vc)::value;
        if constexpr (v < 4) load_to_lds(rsa, a_src[v], dest + at + v * 1024, 0);
        else load_to_lds(rsb, b_src[v - 4], dest + at + HALF + (v - 4) * 1024, 0);
    };
    auto advance = [&]() {
        a_at += 32 * static_cast<size_t>(M);
        b_at += 32 * static_cast<size_t>(N);
        a_left -= 64 * M;
        b_left -= 64 * N;
        if (--load_steps == 0) {
            load_tile += stride;
            open();
        }
    };
    auto next = [](int at) { return at == (RING - 1) * STEP ? 0 : at + STEP; };

    // fragment of the 16-column sub-tile t, half h, of a step: lane = 16 oct + i reads row 8 oct + i / 4
    // (+ 4 h), columns 4 (i % 4) .. + 3
    const int fbase = (8 * oct + (fr >> 2)) * kRow + (fr & 3) * 8;
    int fcol[4];                                                  // sub-tiles 2 u and 2 u + 1
#pragma unroll
    for (int u = 0; u < 4; ++u) fcol[u] = (u ^ (fr >> 2)) * 64 + (oct & 1) * 32;
    u32x4 bf[2][TN], af[2][TM];
    f32x4 acc[TN][TM];
    // read v (0 .. 31) of a step's fragments: B first, halves interleaved
    auto read = [&](auto slotc, auto vc, int at) {
        constexpr int s = decltype(slotc)::value, v = decltype(vc)::value;
        constexpr int t = (v & 15) >> 1, h = v & 1;
        const int from = at + (v < 16 ? HALF + wn * 256 : wm * 256) + h * 4 * kRow + fbase +
                         (fcol[t >> 1] ^ ((t & 1) * 32));
        const u32x2 q = lds_read_tr16(reinterpret_cast<const uint16_t *>(lds + from));
        if constexpr (v < 16) {
            bf[s][t][2 * h] = q[0];
            bf[s][t][2 * h + 1] = q[1];
        } else {
            af[s][t][2 * h] = q[0];
            af[s][t][2 * h + 1] = q[1];
        }
    };
    // instruction n (0 .. 11) of the conversion of a fragment's eight values from fp16 to bf16
    float wide[2];
    auto convert = [&](auto nc, u32x4 &w) {
        constexpr int n = decltype(nc)::value, c = n / 3;
        if constexpr (n % 3 < 2) wide[n % 3] = f16_half_to_f32<n % 3>(w[c]);
        else w[c] = f32x2_to_bf16x2(wide[0], wide[1]);
    };
    using std::integral_constant;
    // The 64 matrix instructions of the step at `at`, beside them the reads of the one behind it and
    // the loads of the fifth one behind it.  A tile's last step leaves its loads to the next tile's first one,
    // since the finished tile passes through its place.
    enum Kind { kFirst, kMiddle, kLast };
    auto step = [&](auto slotc, auto kindc, int at) {
        constexpr int s = decltype(slotc)::value, KIND = decltype(kindc)::value;
        const int ahead = next(at), behind = at == 0 ? (RING - 1) * STEP : at - STEP;
        if constexpr (KIND != kLast) aim();
        static_for<64>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            constexpr int j = m >> 3, i = (j & 1) != 0 ? 7 - (m & 7) : (m & 7);
            mfma_16x16x32_agpr<false, m == 0, KIND == kFirst>(acc[i][j], bf[s][i], af[s][j]);
            if constexpr (m < 32) read(integral_constant<int, 1 - s>{}, mc, ahead);
            if constexpr (KIND == kMiddle && (m & 7) == 7) load(integral_constant<int, j>{}, at);
            if constexpr (KIND == kFirst && (m & 7) >= 6) load(integral_constant<int, 2 * (j & 3) + (m & 1)>{}, m < 32 ? behind : at);
            if constexpr (KIND == kFirst && m == 32) {
                advance();
                aim();
            }
            // the conversion of the next column, of the next step's first in the last one: two of its twelve
            // instructions behind each of six multiplications
            if constexpr (AF16 && (m & 7) < 6) {
                u32x4 &w = j < 7 ? af[s][(j + 1) & 7] : af[1 - s][0];
                convert(integral_constant<int, 2 * (m & 7)>{}, w);
                convert(integral_constant<int, 2 * (m & 7) + 1>{}, w);
            }
            MOE_SB();
        });
        if constexpr (KIND != kLast) advance();
    };
    // In front of step p of a tile: its fragments have been read by every wavefront, so that its place is
    // free, and the step behind it is there.  A tile begins with its first three steps landed, the fourth on its way
    // and, younger than that, up to 64 stores of the tile before.
    auto turn = [&](int p) {
        MOE_SB();
        __builtin_amdgcn_s_waitcnt(0xc07f);      // lgkmcnt(0), in a form that the compiler's own counting sees
        if (p >= 3) MOE_VMCNT(24);               // three steps of loads may be on their way behind that one
        else MOE_VMCNT(63);
        MOE_BAR();
    };
    using S0 = integral_constant<int, 0>;
    using S1 = integral_constant<int, 1>;
    using First = integral_constant<int, kFirst>;
    using Middle = integral_constant<int, kMiddle>;
    using Last = integral_constant<int, kLast>;

    open();
#pragma unroll
    for (int p = 0; p < RING - 1; ++p) {
        aim();
        static_for<8>([&](auto v) { load(v, p * STEP); });
        advance();
    }
    MOE_VMCNT(0);
    MOE_BAR();
    static_for<32>([&](auto v) { read(S0{}, v, 0); });
    if constexpr (AF16) {
#pragma unroll
        for (int c = 0; c < 4; ++c) af[0][0][c] = f16x2_to_bf16x2(af[0][0][c]);
    }
    int at = 0;
    for (; tile < end; tile += stride) {
        const Tile t = tile_at(tile);
        const int steps = t.steps();
        turn(0);
        step(S0{}, First{}, at);
        at = next(at);
        int p = 1;
        for (; p < steps - 1; p += 2) {
            turn(p);
            step(S1{}, Middle{}, at);
            at = next(at);
            turn(p + 1);
            step(S0{}, Middle{}, at);
            at = next(at);
        }
        turn(p);
        step(S1{}, Last{}, at);
        // acc[i][j][c]: column n0 + wn * 128 + i * 16 + oct * 4 + c, row m0 + wm * 128 + j * 16 + fr.  16 rows at a
        // time go through the wavefront's quarter of the last step's place, the 16-byte pieces of a row
        // XOR-swizzled with the row, and leave as two whole rows of 128 columns per instruction.  (LDS takes a
        // wavefront's accesses in order: nothing is waited for in between.)
        MOE_MATRIX_RESULTS();
        MOE_VMCNT(8);
        float *out = C + (static_cast<size_t>(t.expert) * M + t.m0 + wm * 128) * N + t.n0 + wn * 128;
        const __amdgpu_buffer_rsrc_t rsc = __builtin_amdgcn_make_buffer_rsrc(out, 0, 128u * static_cast<unsigned>(N) * 4u, 0x00020000);
        char *const patch = lds + at + wave * 8192;
        const int out_lane = (lane >> 5) * N * 4 + (lane & 31) * 16;
        u32x4 line[2][8];
        auto through = [&](auto jc) {
            constexpr int j = decltype(jc)::value;
#pragma unroll
            for (int i = 0; i < TN; ++i)
                *reinterpret_cast<f32x4 *>(patch + fr * 512 + (((i * 4 + oct) ^ fr) << 4)) = acc[i][j];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int row = 2 * q + (lane >> 5);
                line[j & 1][q] = *reinterpret_cast<const u32x4 *>(patch + row * 512 + (((lane & 31) ^ row) << 4));
            }
            MOE_SB();
        };
        auto leave = [&](auto jc) {
            constexpr int j = decltype(jc)::value;
#pragma unroll
            for (int q = 0; q < 8; ++q)
                __builtin_amdgcn_raw_buffer_store_b128(line[j & 1][q], rsc, out_lane, (j * 16 + 2 * q) * N * 4, 2);
            MOE_SB();
        };
        static_for<TM>([&](auto jc) {
            through(jc);
            if constexpr (decltype(jc)::value > 0) leave(std::integral_constant<int, decltype(jc)::value - 1>{});
        });
        leave(std::integral_constant<int, TM - 1>{});
        at = next(at);
    }
    MOE_VMCNT(0);
}

// ---------------------------------------------------------------- gate backward
// dx[t, i] = sum of the token's kept dxe rows + sum_e dz[e] Wg[i, e], on the fp32 matrix
// instruction (products in ascending e, fused).  Block = 32 tokens x 256 columns, a wavefront 64
// of them: the rows' sums are the accumulators' start, the tokens' dz stay in registers, and
// the packed gate matrix (fp32 [EP][dP], expert-major, zero padded, columns ordered by
// packed_gate_column) is read once per 32 tokens from L2.  Bound by HBM: k fp32 rows in, one out per
// token.  T = 32768, d = 2048, E = 64, k = 2 (0.8 GB), us: 339, and 109 for the logit
// gradients before it; the token-per-wavefront kernel they replace took 800 (LDS reads of the gate
// matrix twice per token).  T = 4096, d = 768, E = 16: 14.3 + 8.6 (23).
template <int NG>
__global__ __launch_bounds__(256) void gate_dx_kernel(
    const float *__restrict__ Wgp, const int32_t *__restrict__ slot_of, const float *__restrict__ dxe,
    const float *__restrict__ dz, float *__restrict__ dx, int t0, int T, int d, int dP, int E, int EP,
    int k, int max_rows)
{   // tokens [t0, T); NG groups of 16 experts
    constexpr int G = 2, CG = 4, NS = NG * 4;
    const int lane = lane_id(), r16 = lane & 15, kq = lane >> 4;
    const int tb = t0 + blockIdx.x * (16 * G);
    const int c0 = blockIdx.y * 256 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * 64;
    if (c0 >= d) return;
    int tok[G];
    float dzr[G][NS];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        tok[g] = min(tb + g * 16 + r16, T - 1);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const float v = dz[static_cast<size_t>(tok[g]) * E + min(4 * s + kq, E - 1)];
            dzr[g][s] = 4 * s + kq < E ? v : 0.0f;
        }
    }
    // (the packed row is padded past d; experts past E: dz is zero)
    const float *wcol = Wgp + c0 + packed_gate_column(r16);
    float wr[CG][NS];
#pragma unroll
    for (int c = 0; c < CG; ++c)
#pragma unroll
        for (int s = 0; s < NS; ++s) wr[c][s] = wcol[static_cast<size_t>(min(4 * s + kq, EP - 1)) * dP + c * 16];
    f32x4 acc[G][CG];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int c = 0; c < CG; ++c) acc[g][c] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 2
    for (int j = 0; j < k; ++j) {
        int slot[G];
        bool kept[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            slot[g] = slot_of[static_cast<size_t>(tok[g]) * k + j];
            kept[g] = slot[g] >= 0 && slot[g] < max_rows;
        }
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int c = 0; c < CG; ++c) {               // (a dropped assignment reads row 0, and drops it)
                const f32x4 v = *reinterpret_cast<const f32x4 *>(
                    dxe + static_cast<size_t>(kept[g] ? slot[g] : 0) * d + min(c0 + c * 16 + 4 * kq, d - 4));
                acc[g][c] += kept[g] ? v : (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
            }
    }
#pragma unroll
    for (int c = 0; c < CG; ++c) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int g = 0; g < G; ++g)
                acc[g][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(wr[c][s], dzr[g][s], acc[g][c], 0, 0, 0);
        // acc[g][c][v]: column c0 + 16 c + 4 kq + v, token tb + 16 g + r16
        const int i = c0 + c * 16 + 4 * kq;
#pragma unroll
        for (int g = 0; g < G; ++g)
            if (i < d && tb + g * 16 + r16 < T)
                *reinterpret_cast<f32x4 *>(dx + static_cast<size_t>(tok[g]) * d + i) = acc[g][c];
    }
}

// partial[s][i][e] = sum over the tokens of range s of x[t, i] dz[t, e], ascending t, on the fp32
// matrix instruction.  Block = 64 columns i (16 per wavefront) x all experts (NG groups of 16);
// tokens go through LDS 64 at a time, the next 64 on their way in registers.  The row pitches (16
// mod 64 words) let the four tokens of an instruction fall into different banks.  T = 32768,
// d = 2048, E = 64, us: 114 (381 with a v_fmac chain per column and a quarter of the experts).
template <int NG>
__global__ __launch_bounds__(256) void dwg_partial_kernel(
    const uint16_t *__restrict__ x, const float *__restrict__ dz, float *__restrict__ partial, int T,
    int d, int E, int per_split)
{
    constexpr int XP = 80, ZP = NG == 1 ? 16 : NG == 2 ? 48 : 80, ZV = NG * 16 * 64 / 256;
    __shared__ __attribute__((aligned(16))) float xs[64 * XP];
    __shared__ float zs[64 * ZP];
    const int tid = threadIdx.x, lane = lane_id(), r16 = lane & 15, kq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i0 = blockIdx.x * 64;
    const int t0 = blockIdx.y * per_split, t1 = min(T, t0 + per_split);
    f32x4 acc[NG];
#pragma unroll
    for (int q = 0; q < NG; ++q) acc[q] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
    u32x4 xr[2];
    float zr[ZV];
    // eight columns per load; what lies past the range or the matrix is zeroed on its way into LDS
    auto load = [&](int tb) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int v = tid + 256 * q;
            xr[q] = *reinterpret_cast<const u32x4 *>(x + static_cast<size_t>(min(tb + v / 8, T - 1)) * d +
                                                     min(i0 + v % 8 * 8, d - 8));
        }
#pragma unroll
        for (int q = 0; q < ZV; ++q) {
            const int v = tid + 256 * q;
            zr[q] = dz[static_cast<size_t>(min(tb + v / (NG * 16), T - 1)) * E + min(v % (NG * 16), E - 1)];
        }
    };
    load(t0);
    for (int tb = t0; tb < t1; tb += 64) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int v = tid + 256 * q, tt = v / 8, c8 = v % 8 * 8;
            const bool in = tb + tt < t1 && i0 + c8 < d;
            f32x4 lo, hi;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                lo[2 * c] = in ? __uint_as_float(xr[q][c] << 16) : 0.0f;
                lo[2 * c + 1] = in ? __uint_as_float(xr[q][c] & 0xFFFF0000u) : 0.0f;
                hi[2 * c] = in ? __uint_as_float(xr[q][2 + c] << 16) : 0.0f;
                hi[2 * c + 1] = in ? __uint_as_float(xr[q][2 + c] & 0xFFFF0000u) : 0.0f;
            }
            *reinterpret_cast<f32x4 *>(xs + tt * XP + c8) = lo;
            *reinterpret_cast<f32x4 *>(xs + tt * XP + c8 + 4) = hi;
        }
#pragma unroll
        for (int q = 0; q < ZV; ++q) {
            const int v = tid + 256 * q, tt = v / (NG * 16), ee = v % (NG * 16);
            zs[tt * ZP + ee] = (tb + tt < t1 && ee < E) ? zr[q] : 0.0f;
        }
        __syncthreads();
        if (tb + 64 < t1) load(tb + 64);
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const float xv = xs[(4 * s + kq) * XP + wave * 16 + r16];
#pragma unroll
            for (int q = 0; q < NG; ++q)
                acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(zs[(4 * s + kq) * ZP + q * 16 + r16], xv, acc[q], 0, 0, 0);
        }
    }
    // acc[q][c]: expert 16 q + 4 kq + c, column i0 + 16 wave + r16
    const int i = i0 + wave * 16 + r16;
    if (i >= d) return;
#pragma unroll
    for (int q = 0; q < NG; ++q)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int e = q * 16 + 4 * kq + c;
            if (e < E) partial[(static_cast<size_t>(blockIdx.y) * d + i) * E + e] = acc[q][c];
        }
}

__global__ void dwg_reduce_kernel(const float *__restrict__ partial, float *__restrict__ dWg, int n,
                                  int splits)
{
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= n) return;
    float acc = 0.0f;
#pragma unroll 8
    for (int s = 0; s < splits; ++s) acc += partial[static_cast<size_t>(s) * n + idx];
    dWg[idx] = acc;
}

// ---------------------------------------------------------------- host side
struct BwdWorkspace {
    Workspace lists;          // work lists of the two row-grouped GEMM shapes
    _Float16 *P;              // [R][h]
    uint16_t *Hb, *dye, *dP;  // [R][h], [R][d], [R][h]
    float *dxe;               // [R][d]
    float *dz, *partial;      // [T][E], [splits][d][E]
    int splits, per_split;
    size_t bytes;
};

// the forward's choice of tile; where the operands are past 32-bit offsets, the general kernel
GemmPlan plan_rows(int N, int K, int64_t max_rows, int E, bool dxe)
{
    GemmPlan gp;
    constexpr uint64_t most = (1ull << 31) - 64;       // byte offsets into the operands and a tile's rows
    if (static_cast<uint64_t>(N) * K * 2 < most && 256ull * K * 2 < most && 256ull * N * 2 < most) {
        choose_w4_tile(max_rows, E, N, K, &gp);
        // (15 training steps of 134 .. 2201 tokens that it takes: 0.93 .. 1.00 of their time, mean 0.97)
        if (dxe && few_long_tiles(max_rows, E, N, K)) {
            gp.bm = gp.bn = 128, gp.concurrent = 32, gp.deep = true;
        }
    } else {
        gp.bm = kBM;
        gp.bn = kBN;
        gp.concurrent = 32;
    }
    gp.tiles_n = (N + gp.bn - 1) / gp.bn;
    gp.max_row_tiles = static_cast<int32_t>((max_rows + gp.bm - 1) / gp.bm + E);
    gp.max_items = work_list_entries(gp);
    return gp;
}

void layout_bwd(const moe_shape &s, void *base, BwdWorkspace *w)
{
    const int64_t R = moe_max_rows(&s);
    char *p = static_cast<char *>(base);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *at = p + off;
        off += align_up(bytes, 256);
        return at;
    };
    w->lists = Workspace{};
    w->lists.gp[0] = plan_rows(s.d_ff, s.d_model, R, s.E, false);
    w->lists.gp[1] = plan_rows(s.d_model, s.d_ff, R, s.E, true);
    for (int g = 0; g < 2; ++g) {      // one list per FFN group of a chunked backward pass
        w->lists.items[g] = reinterpret_cast<WorkItem *>(
            take(sizeof(WorkItem) * w->lists.gp[g].max_items * kMaxChunks));
    }
    const size_t Rh = static_cast<size_t>(R) * s.d_ff, Rd = static_cast<size_t>(R) * s.d_model;
    w->P = reinterpret_cast<_Float16 *>(take(Rh * 2));
    w->Hb = reinterpret_cast<uint16_t *>(take(Rh * 2));
    w->dye = reinterpret_cast<uint16_t *>(take(Rd * 2));
    w->dP = reinterpret_cast<uint16_t *>(take(Rh * 2));
    w->dxe = reinterpret_cast<float *>(take(Rd * 4));
    w->dz = reinterpret_cast<float *>(take(static_cast<size_t>(s.T) * s.E * 4));
    w->splits = std::max(1, std::min(32, (s.T + 127) / 128));
    w->per_split = (s.T + w->splits - 1) / w->splits;
    w->partial = reinterpret_cast<float *>(take(static_cast<size_t>(w->splits) * s.d_model * s.E * 4));
    w->bytes = off;
}

bool supported(const moe_shape *s)
{
    if (s == nullptr || s->dtype != MOE_BF16 || s->renorm_topk != 0) return false;
    if (s->T < 1 || s->d_model < 8 || s->d_ff < 8 || s->E < 1 || s->E > kMaxExperts || s->k < 1 ||
        s->k > kMaxTopK || s->k > s->E || s->capacity < 1)
        return false;
    return s->d_model % 8 == 0 && s->d_ff % 8 == 0;
}

template <int EPI, int ACT, bool KTAIL>
void launch_gemm_k(const uint16_t *A, const uint16_t *W, void *C, _Float16 *P, const WorkItem *items,
                   int N, int K, int grid_items, int stage, hipStream_t st)
{
    auto kern = bwd_gemm_kernel<EPI, ACT, KTAIL>;
    static PerDeviceOnce once;   // raising the dynamic LDS limit: once per kernel and device
    once.raise_lds(reinterpret_cast<const void *>(kern), static_cast<int>(kGemmLds));
    hipEvent_t t0, t1;
    prof_kernel_events(stage, &t0, &t1);
    hipExtLaunchKernelGGL(kern, dim3(grid_items), dim3(512), kGemmLds, st, t0, t1, 0, A, W, C, P, items,
                          N, K);
}

template <int EPI, int ACT>
void launch_gemm(const uint16_t *A, const uint16_t *W, void *C, _Float16 *P, const WorkItem *items,
                 int N, int K, const GemmPlan &gp, int stage, hipStream_t st)
{
    const int grid_items = gp.max_items;
    if (gp.w4) {
        auto launch = [&](auto bm, auto bn, auto tail, auto deep) {
            constexpr int BM = decltype(bm)::value, BN = decltype(bn)::value;
            auto kern = bwd_gemm_w4_kernel<EPI, ACT, decltype(tail)::value, BM, BN, decltype(deep)::value>;
            constexpr size_t lds = decltype(deep)::value ? kW4Lds : w4_lds(BM, BN);
            static PerDeviceOnce once;
            once.raise_lds(reinterpret_cast<const void *>(kern), static_cast<int>(lds));
            hipEvent_t t0, t1;
            prof_kernel_events(stage, &t0, &t1);
            hipExtLaunchKernelGGL(kern, dim3(grid_items), dim3(256), lds, st, t0, t1, 0, A, W, C, P, items,
                                  N, K);
        };
        auto shape = [&](auto tail) {
            using std::integral_constant;
            if (gp.bm == 256)
                launch(integral_constant<int, 256>{}, integral_constant<int, 256>{}, tail, std::false_type{});
            else if (gp.bn == 256)
                launch(integral_constant<int, 128>{}, integral_constant<int, 256>{}, tail, std::false_type{});
            else if (EPI != 0 || !gp.deep)
                launch(integral_constant<int, 128>{}, integral_constant<int, 128>{}, tail, std::false_type{});
            else
                launch(integral_constant<int, 128>{}, integral_constant<int, 128>{}, tail, std::bool_constant<EPI == 0>{});
        };
        if (K % 64 == 0)
            shape(std::false_type{});
        else
            shape(std::true_type{});
        return;
    }
    if (K % kBK != 0)
        launch_gemm_k<EPI, ACT, true>(A, W, C, P, items, N, K, grid_items, stage, st);
    else
        launch_gemm_k<EPI, ACT, false>(A, W, C, P, items, N, K, grid_items, stage, st);
}

// 256 x 256 tiles on four wavefronts when they fit the matrix, there are 512 of them, and the buffer offsets (an expert's
// rows times the row length, in bytes) stay below 2^31.  Time of both gradients / of the training step over that with 128 x
// 128 tiles, 60 layers of 1024 .. 16384 tokens, rows spread evenly; by Zipf(1.2): 512 .. 599 tiles 0.66 .. 0.83 / 0.87 .. 0.88;
// 0.69 .. 0.95 / 0.85 .. 0.89; 640 .. 768 0.73 .. 0.74 / 0.86 .. 0.91; 0.68 .. 0.83 / 0.86 .. 0.88; with every row in one expert 512 .. 1024
// tiles 0.63 .. 1.08 / 0.69 .. 0.95.  On the other side: 360 .. 480 0.66 .. 0.80 / 0.87 .. 0.89; 0.67 .. 0.86 / 0.82 .. 0.91; 288 .. 320
// 0.89 .. 0.93 / 0.76 .. 0.90; 0.83 .. 0.98 / 0.77 .. 0.93; 288 .. 480 with every row in one expert 0.61 .. 0.94 / 0.71 .. 0.94; 160 .. 256 0.65
// .. 0.77 / 0.87 .. 0.92; 0.66 .. 0.99 / 0.85 .. 0.91; one expert 0.62 .. 1.11 / 0.74 .. 1.08; 128 1.02 .. 1.09 / 0.86 .. 1.01; 1.06 .. 1.20
// / 0.88 .. 1.01; 64 1.30 / 1.06; 1.42 / 1.09.  So 512 is on the safe side: it was set for one tile per block, which could take
// 1.6 times as long below it where one expert had most of the rows; shares of the tiles would carry it down to 257.
bool wide_wgrad_tiles(int E, int M, int N, int64_t max_rows)
{
    const uint64_t span = static_cast<uint64_t>(max_rows + 192) * static_cast<uint64_t>(std::max(M, N)) * 2;
    return M % 256 == 0 && N % 256 == 0 && static_cast<int64_t>(E) * (M / 256) * (N / 256) >= 512 && span < (1ull << 31);
}

// dW[e] [M][N] = A[rows of e]^T B[rows of e] from row-major operands
template <bool AF16>
void launch_wgrad(const uint16_t *A, const uint16_t *B, float *C, const int32_t *offsets, int E, int M,
                  int N, int64_t max_rows, int stage, hipStream_t st)
{
    hipEvent_t t0, t1;
    if (wide_wgrad_tiles(E, M, N, max_rows)) {
        constexpr size_t kLds4 = kW4Lds;
        auto kern = wgrad_w4_kernel<AF16>;
        static PerDeviceOnce once;
        once.raise_lds(reinterpret_cast<const void *>(kern), static_cast<int>(kLds4));
        const int tiles_m = M / 256, tiles_n = N / 256;
        // (what leaves of a tile takes as long as five stages)
        const int share = std::max(1, kRunStages / (static_cast<int>((max_rows / E + 63) / 64) + 5));
        const int grid = kRunUnits * ceil_div((E * tiles_m * tiles_n + 7) / 8, kRunUnits / 8 * share);
        prof_kernel_events(stage, &t0, &t1);
        hipExtLaunchKernelGGL(kern, dim3(grid), dim3(256), kLds4, st, t0, t1, 0, A, B, C, offsets, E, M,
                              N, tiles_m, tiles_n, share);
        return;
    }
    constexpr size_t kLds = 2 * 2 * kBK * 128 * sizeof(uint16_t);
    auto kern = wgrad_gemm_kernel<AF16>;
    static PerDeviceOnce once;
    once.raise_lds(reinterpret_cast<const void *>(kern), static_cast<int>(kLds));
    const int tiles_m = (M + 127) / 128, tiles_n = (N + 127) / 128;
    const int grid = static_cast<int>(align_up(static_cast<size_t>(E) * tiles_m * tiles_n, 8));
    prof_kernel_events(stage, &t0, &t1);
    hipExtLaunchKernelGGL(kern, dim3(grid), dim3(256), kLds, st, t0, t1, 0, A, B, C, offsets, E, M, N,
                          tiles_m, tiles_n);
}

// Side streams and events of a chunked backward pass, per device, kept for the process.
struct BwdResources {
    bool ready = false;
    std::mutex enqueue;                 // held while a call enqueues on the side streams
    hipStream_t grad_in = nullptr, grad_out = nullptr;
    hipEvent_t begun = nullptr, joined_in = nullptr, joined_out = nullptr;
    hipEvent_t dispatched[kMaxChunks] = {}, computed[kMaxChunks] = {};
};
std::mutex g_bwd_mutex;
BwdResources g_bwd[16];

moe_status bwd_resources(BwdResources **out)
{
    int dev = 0;
    MOE_TRY_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 16) {
        set_error("device index %d out of range", dev);
        return MOE_EUNSUPPORTED;
    }
    std::lock_guard<std::mutex> lock(g_bwd_mutex);
    BwdResources &r = g_bwd[dev];
    if (!r.ready) {
        MOE_TRY_HIP(hipStreamCreateWithFlags(&r.grad_in, hipStreamNonBlocking));
        MOE_TRY_HIP(hipStreamCreateWithFlags(&r.grad_out, hipStreamNonBlocking));
        MOE_TRY_HIP(hipEventCreateWithFlags(&r.begun, hipEventDisableTiming));
        MOE_TRY_HIP(hipEventCreateWithFlags(&r.joined_in, hipEventDisableTiming));
        MOE_TRY_HIP(hipEventCreateWithFlags(&r.joined_out, hipEventDisableTiming));
        for (int c = 0; c < kMaxChunks; ++c) {
            MOE_TRY_HIP(hipEventCreateWithFlags(&r.dispatched[c], hipEventDisableTiming));
            MOE_TRY_HIP(hipEventCreateWithFlags(&r.computed[c], hipEventDisableTiming));
        }
        r.ready = true;
    }
    *out = &r;
    return MOE_OK;
}

// A side stream and its events for the weight gradients of an unchunked backward pass.  None of the above:
// a chunked pass that is being captured holds those in its capture until the capture ends, and a call
// from outside may neither wait for them nor record on them; these are used outside capture only.  One per
// caller's stream, so that a call does not queue behind another stream's work; a fifth takes over the one
// used longest ago.
struct SideStream {
    hipStream_t caller = nullptr, stream = nullptr;
    hipEvent_t dispatched = nullptr, hidden = nullptr, joined = nullptr;
    uint64_t used = 0;                  // 0: not created yet
};
struct SideStreams {
    std::mutex enqueue;                 // held while a call enqueues on one of them
    uint64_t calls = 0;
    SideStream of[4];
};
SideStreams g_side[16];

// the one of `caller`, created if need be, or NULL; under r.enqueue
SideStream *side_stream(SideStreams &r, hipStream_t caller)
{
    SideStream *s = nullptr;
    for (SideStream &c : r.of)
        if (c.used != 0 && c.caller == caller) s = &c;
    if (s == nullptr) {
        s = &r.of[0];
        for (SideStream &c : r.of)
            if (c.used < s->used) s = &c;
        if (s->used == 0) {
            // (what a call that failed half-way has made is taken over)
            if (s->stream == nullptr && hipStreamCreateWithFlags(&s->stream, hipStreamNonBlocking) != hipSuccess) {
                (void)hipGetLastError();
                return nullptr;
            }
            for (hipEvent_t *e : {&s->dispatched, &s->hidden, &s->joined})
                if (*e == nullptr && hipEventCreateWithFlags(e, hipEventDisableTiming) != hipSuccess) {
                    (void)hipGetLastError();
                    return nullptr;
                }
        }
        s->caller = caller;
    }
    s->used = ++r.calls;
    return s;
}

// Whether an unchunked backward pass runs its weight gradients beside the other GEMMs, which depend on
// them in nothing: each of the four leaves its last round of tiles partly filled, and the gate's
// gradients leave the matrix cores idle.  By `work`, rows x d_model x d_ff: below 2.7e9 the events between
// the streams can cost more than that; in large layers a last round is one of many, and GEMMs that run at
// once share the caches and the power.  us of a training step, one after the other / beside each other, rows spread evenly (by
// Zipf(1.2)), k = 2 unless said.  Below the line: 128 tokens, 8 experts, 256 x 512 68 / 128 (68 / 125); 512, 8, 512 x 1536 115 /
// 128 (115 / 128); 512, 8, 1024 x 2048 182 / 184 (176 / 178); 2048, 16, 512 x 1024 128 / 128 (117 / 127); but 300, 16, 768 x 3072
// (1.4e9) 213 / 210 (214 / 205) and 640, 8, 1024 x 2048 (2.68e9) 179 / 176 (178 / 177).  Above: 1500, 13, 640 x 1536 (2.9e9) 176 / 171
// (162 / 164); 2048, 16, 512 x 1536 172 / 170 (153 / 157); 300, 13, 1536 x 4096 358 / 340 (350 / 331); 8192, 8, 256 x 1024 206 / 182
// (192 / 176); 1024, 16, 768 x 3072 270 / 262 (256 / 244); 4096 of these 457 / 415 (380 / 335); 8192, k = 3 1003 / 945 (814 / 706);
// 4096, 16, 2048 x 8192 2214 / 2128 (1767 / 1616); 32768, 32, 1024 x 4096 3704 / 3705 (2059 / 1996); 16384, 32, 2048 x 8192 (5.5e11)
// 7011 / 6902 (4228 / 3952); 32768, 64, 2048 x 4096 7665 / 7729 (4124 / 3964).  Past it: 24000, 32, 2048 x 8192 (8.1e11) 9541 / 9610
// (5733 / 5339); 32768, 64, 2048 x 8192 (1.1e12) 14032 / 14202 (7447 / 7146).
// Not while the stages are timed, and not under capture: the side stream would stay part of the
// capture after the call returns, when the next call from outside needs it.
bool overlaps_weight_grads(double work, hipStream_t st)
{
    if (work < 2.7e9 || work > 7e11 || prof_enabled()) return false;
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &status) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return status == hipStreamCaptureStatusNone;
}

// The backward pass, cut like the forward: tokens in n_chunks contiguous parts, the row-grouped
// GEMMs once per group of consecutive chunks (ffn_groups).  Gradient rows are dispatched to the
// expert-major order chunk by chunk on one side stream (the backward pass's first all-to-all
// carries them, Sec. 2.2), the two input-gradient GEMMs of a group start when its last chunk is
// there, and the rows that come back are folded into dx chunk by chunk on a second side stream
// (the second all-to-all) while the caller's stream goes on with the next group and then with
// the weight gradients.  Every result is the same bits for every n_chunks.
template <int ACT>
moe_status backward_t(const moe_shape &s, int n_chunks, const uint16_t *x, const float *Wgp,
                      const float *bias, int bias_stride, const uint16_t *W1, const uint16_t *W2,
                      const uint16_t *W1p, const int32_t *expert_idx, const float *gate,
                      const int32_t *offsets, const int32_t *slot_of, const int32_t *src_of,
                      const uint16_t *xe, const _Float16 *ye, const _Float16 *pre,
                      const _Float16 *hid, const float *dy, float *dx, float *dWg, float *dW1,
                      float *dW2, float *dgate, const BwdWorkspace &w, hipStream_t st)
{
    const int T = s.T, d = s.d_model, h = s.d_ff, E = s.E, k = s.k;
    const int R = static_cast<int>(moe_max_rows(&s));
    if (n_chunks > T) n_chunks = T;
    const int n_groups = ffn_groups(s, n_chunks);
    if (n_groups == 1) n_chunks = 1;
    moe_status rc = launch_items(s, n_chunks, n_groups, offsets, src_of, w.lists, st);
    if (rc != MOE_OK) return rc;
    const GemmPlan &g0 = w.lists.gp[0], &g1 = w.lists.gp[1];
    _Float16 *P = pre != nullptr ? const_cast<_Float16 *>(pre) : w.P;
    int EP = 1;
    while (EP < E) EP <<= 1;
    const int NG = EP <= 16 ? 1 : EP / 16;             // groups of 16 experts
    const int dPad = (d + 127) / 128 * 128;            // the packed gate matrix's row length
    auto bound = [&](int c) { return static_cast<int>(static_cast<int64_t>(c) * T / n_chunks); };

    // dye = g dy (bf16) and dgate = <ye, dy> for the tokens [t0, t1)
    auto grad_dispatch = [&](int t0, int t1, hipStream_t q) {
        if (t1 > t0)
            hipLaunchKernelGGL(combine_bwd_kernel, dim3(ceil_div(t1 - t0, 4)), dim3(256), 0, q, dy, ye,
                               slot_of, gate, w.dye, dgate, t0, t1, d, k, R);
    };
    // the row-grouped GEMMs of FFN group f
    auto hidden_grads = [&](int f) {
        const WorkItem *it0 = w.lists.items[0] + static_cast<size_t>(f) * g0.max_items;
        // P = xe W1 (fp16), Hb = act(P) (bf16) -- unless the forward kept P and its hidden activations
        if (pre == nullptr)
            launch_gemm<1, ACT>(xe, W1p, w.Hb, w.P, it0, h, d, g0,
                                kStageBwdRecompute, st);
        // dP = (dye W2^T) * act'(P): W2 [E][h][d] is already "rows n = h, contraction d contiguous"
        launch_gemm<2, ACT>(w.dye, W2, w.dP, P, it0, h, d, g0,
                            kStageBwdDP, st);
    };
    auto input_grads = [&](int f) {
        const WorkItem *it1 = w.lists.items[1] + static_cast<size_t>(f) * g1.max_items;
        // dxe = dP W1^T: W1 [E][d][h] is "rows n = d, contraction h contiguous"
        launch_gemm<0, ACT>(w.dP, W1, w.dxe, nullptr, it1, d, h, g1, kStageBwdDxe,
                            st);
    };
    // dW2[e] [h][d] = act(P)^T dye ; dW1[e] [d][h] = xe^T dP, operands as they are
    auto weight_grad2 = [&](hipStream_t q) {
        if (pre != nullptr)      // the forward's own hidden activations, fp16
            launch_wgrad<true>(reinterpret_cast<const uint16_t *>(hid), w.dye, dW2, offsets, E, h, d, R,
                               kStageBwdWgrad2, q);
        else
            launch_wgrad<false>(w.Hb, w.dye, dW2, offsets, E, h, d, R, kStageBwdWgrad2, q);
    };
    auto weight_grad1 = [&](hipStream_t q) {
        launch_wgrad<false>(xe, w.dP, dW1, offsets, E, d, h, R, kStageBwdWgrad1, q);
    };
    // gate: dz and dx for the tokens [t0, t1)
    moe_status combine_rc = MOE_OK;
    auto grad_combine = [&](int t0, int t1, hipStream_t q) {
        if (t1 <= t0) return;
        const int n = t1 - t0;
        if (combine_rc == MOE_OK)
            combine_rc = launch_gate_grad(s, t0, t1, x, Wgp, bias, bias_stride, expert_idx, dgate, w.dz, q);
#define MOE_GATE_DX_CASE(NG_)                                                                     \
    if (NG == NG_)                                                                                \
        hipLaunchKernelGGL(gate_dx_kernel<NG_>, dim3(ceil_div(n, 32), ceil_div(d, 256)), dim3(256), 0, q, Wgp, \
                           slot_of, w.dxe, w.dz, dx, t0, t1, d, dPad, E, EP, k, R);
        MOE_GATE_DX_CASE(1) MOE_GATE_DX_CASE(2) MOE_GATE_DX_CASE(4)
#undef MOE_GATE_DX_CASE
    };
    // dWg = x^T dz: partial sums over fixed token ranges, then a fixed-order sum
    auto gate_weight_grad = [&]() {
#define MOE_DWG_CASE(NG_)                                                                         \
    if (NG == NG_)                                                                                \
        hipLaunchKernelGGL(dwg_partial_kernel<NG_>, dim3(ceil_div(d, 64), w.splits), dim3(256), 0, \
                           st, x, w.dz, w.partial, T, d, E, w.per_split);
        MOE_DWG_CASE(1) MOE_DWG_CASE(2) MOE_DWG_CASE(4)
#undef MOE_DWG_CASE
        hipLaunchKernelGGL(dwg_reduce_kernel, dim3(ceil_div(d * E, 256)), dim3(256), 0, st, w.partial,
                           dWg, d * E, w.splits);
    };

    if (n_chunks == 1) {
        SideStream *side = nullptr;
        std::unique_lock<std::mutex> enqueue;
        int dev = 0;
        if (overlaps_weight_grads(static_cast<double>(R) * d * h, st) && hipGetDevice(&dev) == hipSuccess &&
            dev >= 0 && dev < 16) {
            enqueue = std::unique_lock<std::mutex>(g_side[dev].enqueue);
            side = side_stream(g_side[dev], st);
        }
        if (side == nullptr) {
            if (enqueue.owns_lock()) enqueue.unlock();
            grad_dispatch(0, T, st);
            hidden_grads(0);
            input_grads(0);
            weight_grad2(st);
            weight_grad1(st);
            grad_combine(0, T, st);
            gate_weight_grad();
            MOE_TRY_HIP(hipGetLastError());
            return combine_rc;
        }
        count_path_call(kPathSideWeightGrads);
        // The two weight gradients on a side stream: dW2 beside dP from dye on, dW1 beside dxe and the
        // gate's gradients from dP on.
        auto enqueue_both = [&]() -> moe_status {
            grad_dispatch(0, T, st);
            MOE_TRY_HIP(hipEventRecord(side->dispatched, st));
            hidden_grads(0);
            MOE_TRY_HIP(hipEventRecord(side->hidden, st));
            // (dW2 reads the hidden activations: where they are recomputed, the first of the hidden_grads
            // GEMMs writes them)
            MOE_TRY_HIP(hipStreamWaitEvent(side->stream, pre != nullptr ? side->dispatched : side->hidden, 0));
            weight_grad2(side->stream);
            input_grads(0);
            MOE_TRY_HIP(hipStreamWaitEvent(side->stream, side->hidden, 0));
            weight_grad1(side->stream);
            grad_combine(0, T, st);
            gate_weight_grad();
            return MOE_OK;
        };
        rc = enqueue_both();
        // (joined also after a failure part-way)
        hipError_t je = hipEventRecord(side->joined, side->stream);
        if (je == hipSuccess) je = hipStreamWaitEvent(st, side->joined, 0);
        if (rc != MOE_OK) return rc;
        if (je != hipSuccess) return hip_fail(je, "joining the side stream");
        MOE_TRY_HIP(hipGetLastError());
        return combine_rc;
    }

    BwdResources *r = nullptr;
    rc = bwd_resources(&r);
    if (rc != MOE_OK) return rc;
    std::lock_guard<std::mutex> enqueue(r->enqueue);
    MOE_TRY_HIP(hipEventRecord(r->begun, st));
    MOE_TRY_HIP(hipStreamWaitEvent(r->grad_in, r->begun, 0));
    MOE_TRY_HIP(hipStreamWaitEvent(r->grad_out, r->begun, 0));
    auto enqueue_chunks = [&]() -> moe_status {
        for (int c = 0; c < n_chunks; ++c) {
            grad_dispatch(bound(c), bound(c + 1), r->grad_in);
            MOE_TRY_HIP(hipEventRecord(r->dispatched[c], r->grad_in));
        }
        for (int f = 0; f < n_groups; ++f) {
            const int c0 = static_cast<int>(static_cast<int64_t>(f) * n_chunks / n_groups);
            const int c1 = static_cast<int>(static_cast<int64_t>(f + 1) * n_chunks / n_groups);
            MOE_TRY_HIP(hipStreamWaitEvent(st, r->dispatched[c1 - 1], 0));
            hidden_grads(f);
            input_grads(f);
            MOE_TRY_HIP(hipEventRecord(r->computed[f], st));
            MOE_TRY_HIP(hipStreamWaitEvent(r->grad_out, r->computed[f], 0));
            for (int c = c0; c < c1; ++c) grad_combine(bound(c), bound(c + 1), r->grad_out);
        }
        weight_grad2(st);
        weight_grad1(st);
        return MOE_OK;
    };
    rc = enqueue_chunks();
    // join both side streams (also after a failure part-way), then the gate matrix's gradient,
    // which needs every token's dz
    hipError_t je = hipEventRecord(r->joined_in, r->grad_in);
    if (je == hipSuccess) je = hipStreamWaitEvent(st, r->joined_in, 0);
    if (je == hipSuccess) je = hipEventRecord(r->joined_out, r->grad_out);
    if (je == hipSuccess) je = hipStreamWaitEvent(st, r->joined_out, 0);
    if (rc != MOE_OK) return rc;
    if (je != hipSuccess) return hip_fail(je, "joining the side streams");
    gate_weight_grad();
    MOE_TRY_HIP(hipGetLastError());
    return combine_rc;
}

}  // namespace
}  // namespace moe

using namespace moe;

extern "C" {

moe_status moe_backward_gemm_kernel(const moe_shape *s, int32_t which, char *name, size_t len)
{
    if (!supported(s) || name == nullptr || len == 0 || which < 0 || which > 3) {
        set_error("moe_backward_gemm_kernel: which must be in 0..3, name a buffer, the shape one that moe_layer_backward takes");
        return MOE_EINVAL;
    }
    const int64_t R = moe_max_rows(s);
    const int d = s->d_model, h = s->d_ff;
    if (which < 2) {
        const GemmPlan gp = which == 0 ? plan_rows(h, d, R, s->E, false) : plan_rows(d, h, R, s->E, true);
        std::snprintf(name, len, "%s %dx%d%s", gp.w4 ? "bwd_gemm_w4_kernel" : "bwd_gemm_kernel", gp.bm, gp.bn, gp.deep ? " deep" : "");
    } else {
        std::snprintf(name, len, "%s", wide_wgrad_tiles(s->E, which == 2 ? h : d, which == 2 ? d : h, R)
                                           ? "wgrad_w4_kernel 256x256" : "wgrad_gemm_kernel 128x128");
    }
    return MOE_OK;
}

size_t moe_backward_workspace_bytes(const moe_shape *s)
{
    if (!supported(s)) return 0;
    BwdWorkspace w;
    layout_bwd(*s, reinterpret_cast<void *>(static_cast<uintptr_t>(256)), &w);   // sizes only
    return w.bytes;
}

moe_status moe_layer_backward(const moe_shape *s, const void *x, const void *Wgp,
                              const float *gate_bias, int32_t bias_token_stride,
                              const void *W1, const void *W2, const void *W1p,
                              const int32_t *expert_idx, const float *gate,
                              const int32_t *offsets, const int32_t *slot_of,
                              const int32_t *src_of, const void *xe, const void *ye,
                              const void *pre, const void *hid, const float *dy, float *dx,
                              float *dWg, float *dW1, float *dW2, float *dgate, void *workspace,
                              void *stream)
{
    return moe_layer_backward_chunked(s, 1, x, Wgp, gate_bias, bias_token_stride, W1, W2, W1p,
                                      expert_idx, gate, offsets, slot_of, src_of, xe, ye, pre, hid, dy,
                                      dx, dWg, dW1, dW2, dgate, workspace, stream);
}

moe_status moe_layer_backward_chunked(const moe_shape *s, int32_t n_chunks, const void *x,
                                      const void *Wgp, const float *gate_bias,
                                      int32_t bias_token_stride, const void *W1, const void *W2,
                                      const void *W1p, const int32_t *expert_idx, const float *gate,
                                      const int32_t *offsets, const int32_t *slot_of,
                                      const int32_t *src_of, const void *xe, const void *ye,
                                      const void *pre, const void *hid, const float *dy, float *dx,
                                      float *dWg, float *dW1, float *dW2, float *dgate,
                                      void *workspace, void *stream)
{
    if (!supported(s)) {
        set_error("moe_layer_backward: bf16 layers without top-k renormalisation only, E <= %d, "
                  "k <= %d, d_model and d_ff multiples of 8", kMaxExperts, kMaxTopK);
        return s == nullptr ? MOE_EINVAL : MOE_EUNSUPPORTED;
    }
    if (gate_bias != nullptr && bias_token_stride != 0 && bias_token_stride != s->E) {
        set_error("bias_token_stride must be 0 or E");
        return MOE_EINVAL;
    }
    if (n_chunks < 1 || n_chunks > kMaxChunks) {
        set_error("n_chunks must be in 1..%d, got %d", kMaxChunks, n_chunks);
        return MOE_EINVAL;
    }
    const void *need[] = {x, Wgp, W1, W2, W1p, expert_idx, gate, offsets, slot_of, src_of, xe, ye, dy,
                          dx, dWg, dW1, dW2, dgate, workspace};
    for (const void *p : need) {
        if (p == nullptr || (reinterpret_cast<uintptr_t>(p) & 15u) != 0) {
            set_error("moe_layer_backward: a required pointer is NULL or not 16-byte aligned");
            return MOE_EINVAL;
        }
    }
    if (((reinterpret_cast<uintptr_t>(pre) | reinterpret_cast<uintptr_t>(hid)) & 15u) != 0 ||
        (pre == nullptr) != (hid == nullptr)) {
        set_error("moe_layer_backward: pre and hid come together (both or neither), 16-byte aligned");
        return MOE_EINVAL;
    }
    BwdWorkspace w;
    layout_bwd(*s, workspace, &w);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const _Float16 *preh = static_cast<const _Float16 *>(pre);
    const _Float16 *hidh = static_cast<const _Float16 *>(hid);
    const uint16_t *xb = static_cast<const uint16_t *>(x);
    const float *Wgf = static_cast<const float *>(Wgp);
    const uint16_t *W1b = static_cast<const uint16_t *>(W1), *W2b = static_cast<const uint16_t *>(W2);
    const uint16_t *W1pb = static_cast<const uint16_t *>(W1p), *xeb = static_cast<const uint16_t *>(xe);
#define MOE_BWD_CASE(ACT)                                                                         \
    case ACT:                                                                                     \
        return backward_t<ACT>(*s, n_chunks, xb, Wgf, gate_bias, bias_token_stride, W1b, W2b, W1pb, \
                               expert_idx, gate, offsets, slot_of, src_of, xeb,                   \
                               static_cast<const _Float16 *>(ye), preh, hidh,                     \
                               dy, dx, dWg, dW1, dW2, dgate, w, st);
    switch (s->act) {
        MOE_BWD_CASE(MOE_ACT_GELU_ERF)
        MOE_BWD_CASE(MOE_ACT_GELU_TANH)
        MOE_BWD_CASE(MOE_ACT_RELU)
        MOE_BWD_CASE(MOE_ACT_IDENTITY)
    }
#undef MOE_BWD_CASE
    set_error("unknown activation %d", static_cast<int>(s->act));
    return MOE_EINVAL;
}

}  // extern "C"
