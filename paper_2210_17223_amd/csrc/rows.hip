// Row movers: pack tokens into the expert-major buffer (the payload of the first
// all-to-all, paper end of Sec. 2.1) and the gate-weighted unpack ("combine",
// Sec. 2.2 forward-pass timeline).  Both are bound by HBM bandwidth: one wavefront
// owns one token, every lane moves 16 bytes per step, a token's row is read once
// and written to each of its kept slots (pack) or its kept expert rows are read
// once and the weighted sum written once (unpack).  Expert outputs are stored in fp16 for
// bf16 layers (fp32 for fp32 layers); the weighted sum and y are fp32.
#include "common.h"

#include <algorithm>
#include <type_traits>

namespace moe {
namespace {

constexpr int kRowWaves = 4;
constexpr int kRowThreads = kRowWaves * kWave;

// xe[slot_of[t*k+j], :] = x[t, :] for kept j.  `vec` = 16-byte vectors per row.
__global__ __launch_bounds__(kRowThreads) void scatter_rows_kernel(
    const uint4 *__restrict__ x, const int32_t *__restrict__ slot_of,
    uint4 *__restrict__ xe, int t0, int t1, int k, int vec, int max_rows)
{
    const int lane = lane_id();
    const int t = t0 + blockIdx.x * kRowWaves + threadIdx.x / kWave;
    if (t >= t1) return;
    int my_slot = lane < k ? slot_of[static_cast<size_t>(t) * k + lane] : -1;
    if (my_slot >= max_rows) my_slot = -1;   // never follow a slot outside the buffer
    const uint64_t kept = __ballot(my_slot >= 0);
    if (kept == 0) return;
    int slots[kMaxTopK];
#pragma unroll
    for (int j = 0; j < kMaxTopK; ++j) slots[j] = __shfl(my_slot, j);
    const uint4 *src = x + static_cast<size_t>(t) * vec;
    for (int c = lane; c < vec; c += kWave) {
        const uint4 v = src[c];
#pragma unroll
        for (int j = 0; j < kMaxTopK; ++j)
            if (j < k && slots[j] >= 0) xe[static_cast<size_t>(slots[j]) * vec + c] = v;
    }
}

// y[t,:] = sum_j gate[t,j] * ye[slot_of[t*k+j],:] over kept j, ascending j, in fp32.
// TIn: stored type of the expert outputs (fp16 for bf16 layers, fp32 for fp32 layers); a lane
// takes 16 bytes of every kept row per step (NV = 8 or 4 elements) and writes NV fp32 values.
// ACT_BYTES: element size of the optional copy in the activation dtype (0 = none).
// A wavefront owns a token's vectors [blockIdx.y * 64 U, + 64 U); K: k where it is 1 or 2, else 0.
// The loads of all U steps (and both rows where K = 2) are in flight together.
// Few tokens are spread over more wavefronts (small U), many get more loads per wavefront (U = 4: 2 takes
// 102 us in the last of these).  us, with one wavefront per token, one step after the other / so: 256 x 4096
// with the 16-bit copy 10.2 / 5.2; 4096 x 768 6.4 / 6.6; 16384 x 1024 25.5 / 22.9; 32768 x 2048 95 / 86.5.
template <typename TIn, int ACT_BYTES, int U, int K>
__global__ __launch_bounds__(kRowThreads) void combine_rows_kernel(
    const uint4 *__restrict__ ye, const int32_t *__restrict__ slot_of,
    const float *__restrict__ gate, float *__restrict__ y, void *__restrict__ y_act,
    int t0, int t1, int k, int vec, int max_rows)
{
    constexpr int NV = 16 / static_cast<int>(sizeof(TIn)), KM = K != 0 ? K : kMaxTopK;
    const int lane = lane_id();
    const int t = t0 + blockIdx.x * kRowWaves + threadIdx.x / kWave;
    if (t >= t1) return;
    if constexpr (K != 0) k = K;
    int my_slot = lane < k ? slot_of[static_cast<size_t>(t) * k + lane] : -1;
    if (my_slot >= max_rows) my_slot = -1;   // never follow a slot outside the buffer
    const float my_gate = lane < k ? gate[static_cast<size_t>(t) * k + lane] : 0.0f;
    // (one pass but for rows of more pieces than a grid has)
    for (int c0 = blockIdx.y * (kWave * U) + lane; c0 - lane < vec; c0 += gridDim.y * (kWave * U)) {
        float acc[U][NV];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < NV; ++i) acc[u][i] = 0.0f;
        bool first = true;
        auto load = [&](uint4 (&raw)[U], int slot) {
#pragma unroll
            for (int u = 0; u < U; ++u)              // (past the row's end: its last vector, not stored)
                raw[u] = ye[static_cast<size_t>(slot) * vec + min(c0 + u * kWave, vec - 1)];
        };
        auto add = [&](const uint4 (&raw)[U], float g) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float v[NV];
                if constexpr (NV == 8) {
                    typedef __attribute__((ext_vector_type(8))) _Float16 half8;
                    const half8 hv = __builtin_bit_cast(half8, raw[u]);
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = static_cast<float>(hv[i]);
                } else {
                    v[0] = __uint_as_float(raw[u].x); v[1] = __uint_as_float(raw[u].y);
                    v[2] = __uint_as_float(raw[u].z); v[3] = __uint_as_float(raw[u].w);
                }
#pragma unroll
                for (int i = 0; i < NV; ++i) acc[u][i] = first ? g * v[i] : __builtin_fmaf(g, v[i], acc[u][i]);
            }
            first = false;
        };
        if constexpr (K == 2) {
            const int s0 = __shfl(my_slot, 0), s1 = __shfl(my_slot, 1);
            uint4 a[U], b[U];
            if (s0 >= 0) load(a, s0);
            if (s1 >= 0) load(b, s1);
            if (s0 >= 0) add(a, __shfl(my_gate, 0));
            if (s1 >= 0) add(b, __shfl(my_gate, 1));
        } else {
            for (int j = 0; j < KM; ++j) {
                if (j >= k) break;
                const int slot = __shfl(my_slot, j);
                if (slot < 0) continue;
                uint4 raw[U];
                load(raw, slot);
                add(raw, __shfl(my_gate, j));
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = c0 + u * kWave;
            if (c >= vec) break;
            const size_t at = (static_cast<size_t>(t) * vec + c) * NV;       // element index in the row-major output
#pragma unroll
            for (int i = 0; i < NV; i += 4)
                *reinterpret_cast<float4 *>(y + at + i) = make_float4(acc[u][i], acc[u][i + 1], acc[u][i + 2], acc[u][i + 3]);
            if constexpr (ACT_BYTES == 4) {
#pragma unroll
                for (int i = 0; i < NV; i += 4)
                    *reinterpret_cast<float4 *>(static_cast<float *>(y_act) + at + i) =
                        make_float4(acc[u][i], acc[u][i + 1], acc[u][i + 2], acc[u][i + 3]);
            } else if constexpr (ACT_BYTES == 2) {
                uint32_t p[NV / 2];
#pragma unroll
                for (int i = 0; i < NV; i += 2)
                    p[i / 2] = f32_to_bf16(acc[u][i]) | (static_cast<uint32_t>(f32_to_bf16(acc[u][i + 1])) << 16);
                if constexpr (NV == 8)
                    *reinterpret_cast<uint4 *>(static_cast<uint16_t *>(y_act) + at) = make_uint4(p[0], p[1], p[2], p[3]);
                else
                    *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(y_act) + at) = make_uint2(p[0], p[1]);
            }
        }
    }
}

}  // namespace

moe_status launch_scatter(const moe_shape &s, const void *x, const int32_t *slot_of,
                          void *xe, int t0, int t1, hipStream_t st)
{
    if (t1 <= t0) return MOE_OK;
    const int elem = s.dtype == MOE_BF16 ? 2 : 4;
    const int max_rows = static_cast<int>(moe_max_rows(&s));
    const int vec = s.d_model * elem / 16;
    hipLaunchKernelGGL(scatter_rows_kernel, dim3(ceil_div(t1 - t0, kRowWaves)),
                       dim3(kRowThreads), 0, st, static_cast<const uint4 *>(x), slot_of,
                       static_cast<uint4 *>(xe), t0, t1, s.k, vec, max_rows);
    MOE_TRY_HIP(hipGetLastError());
    return MOE_OK;
}

moe_status launch_combine(const moe_shape &s, const void *ye, const int32_t *slot_of,
                          const float *gate, float *y, void *y_act, int t0, int t1,
                          hipStream_t st, int64_t rows)
{
    if (t1 <= t0) return MOE_OK;
    const int vec = s.d_model * ye_elem_bytes(s) / 16;   // 16-byte vectors per row of ye
    const int max_rows = static_cast<int>(rows < 0 ? moe_max_rows(&s) : rows);
    const uint4 *ye4 = static_cast<const uint4 *>(ye);
    const int64_t steps = static_cast<int64_t>(t1 - t0) * ((vec + kWave - 1) / kWave);   // of 64 vectors
    auto launch = [&](auto in, auto act, auto u_, auto k_) {
        constexpr int U = decltype(u_)::value;
        hipLaunchKernelGGL((combine_rows_kernel<decltype(in), decltype(act)::value, U, decltype(k_)::value>),
                           dim3(ceil_div(t1 - t0, kRowWaves), std::min(ceil_div(vec, kWave * U), 65535)), dim3(kRowThreads), 0, st,
                           ye4, slot_of, gate, y, y_act, t0, t1, s.k, vec, max_rows);
    };
    auto with_k = [&](auto in, auto act, auto u_) {
        if (s.k == 1)
            launch(in, act, u_, std::integral_constant<int, 1>{});
        else if (s.k == 2)
            launch(in, act, u_, std::integral_constant<int, 2>{});
        else
            launch(in, act, u_, std::integral_constant<int, 0>{});
    };
    auto with_u = [&](auto in, auto act) {
        if (steps <= 4096)
            with_k(in, act, std::integral_constant<int, 1>{});
        else if (vec < 4 * kWave || steps <= 65536)
            with_k(in, act, std::integral_constant<int, 2>{});
        else
            with_k(in, act, std::integral_constant<int, 4>{});
    };
    if (s.dtype == MOE_BF16) {
        if (y_act == nullptr)
            with_u(_Float16{}, std::integral_constant<int, 0>{});
        else
            with_u(_Float16{}, std::integral_constant<int, 2>{});
    } else {
        if (y_act == nullptr)
            with_u(float{}, std::integral_constant<int, 0>{});
        else
            with_u(float{}, std::integral_constant<int, 4>{});
    }
    MOE_TRY_HIP(hipGetLastError());
    return MOE_OK;
}

}  // namespace moe
