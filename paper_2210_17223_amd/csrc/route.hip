// Gate: logits, top-k selection and softmax gate weights (paper Sec. 2.1).
//
// The logit of (token, expert) is one fp32 accumulator walked over the model
// dimension in ascending order with fused multiply-adds, so that the top-k
// decision (an integer result) does not depend on a reduction tree.
#include "common.h"

#include <type_traits>

namespace moe {
namespace {

constexpr int kGatePad = 128; // the packed gate matrix pads the model dimension to this
constexpr int kKC = 64;       // model-dimension columns per stage

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;

// Top-k, softmax weights and the histogram of a block's tokens from their logits in LDS
// (zs[token][expert]; the histogram sits behind them), with LP lanes per token -- all 256
// lanes when the block has few tokens: lane `sub` of a token's group holds the logits of
// experts sub, sub + LP, ... (NQ of them) in registers; maxima, sums and the k selections
// are butterflies over the group.  Groups are aligned pieces of one wavefront.
template <int NQ, int LP, int TB>
__device__ __forceinline__ void route_tail(float (*zs)[kMaxExperts + 1], int32_t *__restrict__ expert_idx,
                                           float *__restrict__ gate, int32_t *__restrict__ seg_cnt,
                                           int t0, int T, int E, int k, int renorm)
{
    const int tid = threadIdx.x;
    int32_t *cnt = reinterpret_cast<int32_t *>(&zs[kWave][0]);
    if (seg_cnt != nullptr && tid < kMaxExperts) cnt[tid] = 0;
    const int tl = tid / LP, sub = tid % LP;
    const int t = t0 + tl;
    const bool live = tl < TB && t < T;
    float zl[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int e = sub + LP * q;
        zl[q] = (live && e < E) ? zs[tl][e] : -INFINITY;
    }
    if (seg_cnt != nullptr) __syncthreads();     // the histogram is cleared
    float zmax = zl[0];
#pragma unroll
    for (int q = 1; q < NQ; ++q) zmax = fmaxf(zmax, zl[q]);
#pragma unroll
    for (int m = 1; m < LP; m <<= 1) zmax = fmaxf(zmax, __shfl_xor(zmax, m));
    float denom = 0.0f;
#pragma unroll
    for (int q = 0; q < NQ; ++q)
        if (sub + LP * q < E) denom += expf(zl[q] - zmax);
#pragma unroll
    for (int m = 1; m < LP; m <<= 1) denom += __shfl_xor(denom, m);

    constexpr int kNone = 0x7fffffff;            // "no candidate": never wins a comparison
    float sel_z[kMaxTopK];
    int sel_e[kMaxTopK];
    uint32_t taken = 0;                          // bit q: this lane's q-th expert is selected
    float gsum = 0.0f;
#pragma unroll
    for (int j = 0; j < kMaxTopK; ++j) {
        sel_z[j] = 0.0f;
        sel_e[j] = 0;
        if (j < k) {
            float bz = -INFINITY;
            int be = kNone;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int e = sub + LP * q;      // ascending in q: a strict > keeps the lower index
                if (e < E && !((taken >> q) & 1u) && (be == kNone || zl[q] > bz)) {
                    bz = zl[q];
                    be = e;
                }
            }
#pragma unroll
            for (int m = 1; m < LP; m <<= 1) {
                const float oz = __shfl_xor(bz, m);
                const int oe = __shfl_xor(be, m);
                if (oe != kNone && (be == kNone || oz > bz || (oz == bz && oe < be))) {
                    bz = oz;
                    be = oe;
                }
            }
            if (be != kNone && be % LP == sub) taken |= 1u << (be / LP);
            sel_z[j] = bz;
            sel_e[j] = be;
            gsum += expf(bz - zmax) / denom;
        }
    }
    if (live && sub == 0) {
#pragma unroll
        for (int j = 0; j < kMaxTopK; ++j) {
            if (j < k) {
                const float g = expf(sel_z[j] - zmax) / denom;
                expert_idx[static_cast<size_t>(t) * k + j] = sel_e[j];
                gate[static_cast<size_t>(t) * k + j] = renorm ? g / gsum : g;
                if (seg_cnt != nullptr) atomicAdd(&cnt[sel_e[j]], 1);
            }
        }
    }
    if (seg_cnt != nullptr) {
        __syncthreads();
        if (tid < kMaxExperts)
            seg_cnt[static_cast<size_t>(blockIdx.x) * kMaxExperts + tid] = cnt[tid];
    }
}

// What a block does with its tokens' logits: the gate's decision, or the gradient of the logits.
struct RouteTail {
    int32_t *expert_idx;
    float *gate;
    int32_t *seg_cnt;
    int k, renorm;
    template <int NQ, int LP, int TB>
    __device__ __forceinline__ void run(float (*zs)[kMaxExperts + 1], int t0, int T, int E) const
    {
        route_tail<NQ, LP, TB>(zs, expert_idx, gate, seg_cnt, t0, T, E, k, renorm);
    }
};

// dz = p (dg - <p, dg>) with p the softmax of the logits and dg the gradient of the selected gate
// weights (zero elsewhere); lanes as in route_tail.
struct GateGradTail {
    const int32_t *expert_idx;
    const float *dgate;
    float *dz;
    int k;
    template <int NQ, int LP, int TB>
    __device__ __forceinline__ void run(float (*zs)[kMaxExperts + 1], int t0, int T, int E) const
    {
        const int tl = threadIdx.x / LP, sub = threadIdx.x % LP;
        const int t = t0 + tl;
        const bool live = tl < TB && t < T;
        float p[NQ], dg[NQ], zmax = -INFINITY;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            p[q] = (live && sub + LP * q < E) ? zs[tl][sub + LP * q] : -INFINITY;
            dg[q] = 0.0f;
            zmax = fmaxf(zmax, p[q]);
        }
#pragma unroll
        for (int m = 1; m < LP; m <<= 1) zmax = fmaxf(zmax, __shfl_xor(zmax, m));
        if (live)
            for (int j = 0; j < k; ++j) {
                const int e = expert_idx[static_cast<size_t>(t) * k + j];
                const float g = dgate[static_cast<size_t>(t) * k + j];
#pragma unroll
                for (int q = 0; q < NQ; ++q)
                    if (e == sub + LP * q) dg[q] = g;
            }
        float denom = 0.0f, s = 0.0f;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            p[q] = sub + LP * q < E ? expf(p[q] - zmax) : 0.0f;
            denom += p[q];
        }
#pragma unroll
        for (int m = 1; m < LP; m <<= 1) denom += __shfl_xor(denom, m);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            p[q] /= denom;
            s += p[q] * dg[q];
        }
#pragma unroll
        for (int m = 1; m < LP; m <<= 1) s += __shfl_xor(s, m);
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            if (live && sub + LP * q < E) dz[static_cast<size_t>(t) * E + sub + LP * q] = p[q] * (dg[q] - s);
    }
};

// Logits on the fp32 matrix instruction.  v_mfma_f32_16x16x4_f32 adds its four products to the
// accumulator one after the other in ascending k, each as a fused multiply-add: a chain of
// these instructions over the model dimension is the chain of d fused multiply-adds the gate
// is defined by, bit for bit (denormals included: the test of the gate's logits), for
// 16 tokens x 16 experts at once.  A dependent chain advances one column in 8 cycles (10 for
// v_fmac) and the instruction does 32 multiply-adds per cycle and SIMD (16 for v_fmac).
//
// Block = TB tokens x all experts (padded to EG groups of 16): NC wavefronts multiply -- TB / 16
// token groups, the expert groups spread over up to four wavefronts -- and NL wavefronts bring
// the operands, because any vector instruction between two dependent matrix instructions
// costs the chain 18 cycles on top of its 32 (measured; LDS reads cost it nothing).  The
// loading wavefronts keep PD 64-column stages of global loads in flight in registers, convert
// to fp32 and write LDS tiles in the order the matrix instruction wants its operands: one
// 16-byte read gives a lane its values of four steps.  A lane needs column 4 i + lane / 16 of
// step i; a tile of 16 rows is [quad of steps][lane / 16][row] of 16 bytes with a pitch of 272
// bytes per 16-lane group, which keeps both the reads and the writes free of bank conflicts.
// (The packed gate matrix has a lane's four columns side by side: regrouped on the way instead,
// by 4-byte LDS writes or 4-byte loads, 64 experts took a tenth / a third longer at T = 32768, d = 2048.)
// Three stages of tiles: one barrier per stage, in
// the middle of the multipliers' stage, so that their reads run on across stage boundaries.
//
// Few tokens: bound by the chain (3.3 ns per column at 2.4 GHz), so blocks hold as few tokens
// as the matrix instruction allows.  Many: bound by the matrix cores (T d E / 78.6e12 s) or by
// reading x.  Measured against one v_fmac chain per lane or a register block of them (us, alone):
// T = 4096, d = 768, E = 16: 8.5 (11.6); 256, 4096, 8: 21.1 (34.2); 3001, 1000, 13: 9.4 (18.3);
// 16384, 1024, 32: 18.8 (31.3); 32768, 2048, 64: 100 (148; 105 - 116 inside a layer, where GEMMs of
// milliseconds have set the clock).
template <typename XT, int TB, int EG>
struct RouteTile {
    static constexpr int TG = TB / 16;                       // token groups
    static constexpr int WE = 4 / TG;                        // wavefronts side by side over experts, at most
    static constexpr int NACC = (EG + WE - 1) / WE;          // expert groups per wavefront
    static constexpr int NC = TG * (EG / NACC);              // wavefronts that multiply
    static constexpr int NL = NC < 3 ? 4 - NC : 4;           // ... that load
    static constexpr int NT = (NC + NL) * 64;
    static constexpr int XV = 64 * static_cast<int>(sizeof(XT)) / 16;       // 16-byte vectors per token row and stage
    static constexpr int VECS = TB * XV + EG * 16 * 16;
    static constexpr int VPT = (VECS + NL * 64 - 1) / (NL * 64);            // ... per loading thread
    static constexpr int PD = VPT <= 2 ? 6 : VPT <= 3 ? 4 : VPT <= 6 ? 3 : 2;   // stages in flight in registers
    static constexpr int GROUP = 272, QUAD = 4 * GROUP;      // bytes per 16-lane group, and of a 16-row tile's quad
    static constexpr int TILE = 4 * QUAD, STAGE = (TG + EG) * TILE;
    static constexpr size_t LOGITS = sizeof(float) * (kWave + 2) * (kMaxExperts + 1);
    static constexpr size_t LDS = 3 * static_cast<size_t>(STAGE) > LOGITS ? 3 * static_cast<size_t>(STAGE) : LOGITS;
};

template <typename XT, int TB, int EG, typename Tail>
__global__ __launch_bounds__((RouteTile<XT, TB, EG>::NT), 1) void route_mfma_kernel(
    const XT *__restrict__ x, const float *__restrict__ Wgp, const float *__restrict__ bias,
    int bias_stride, Tail tail, int T, int d, int dP, int E, int EP)
{
    using RT = RouteTile<XT, TB, EG>;
    constexpr int NACC = RT::NACC, TG = RT::TG, NC = RT::NC, STAGE = RT::STAGE, TILE = RT::TILE;
    constexpr int QUAD = RT::QUAD, GROUP = RT::GROUP;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    char *tiles = reinterpret_cast<char *>(smem);
    float (*zs)[kMaxExperts + 1] = reinterpret_cast<float (*)[kMaxExperts + 1]>(smem);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t0 = blockIdx.x * TB;
    const int nstage = (d + kKC - 1) / kKC;           // (columns past d meet zeros of the matrix)
    const int r16 = lane & 15, kq = lane >> 4;
    const int tg = wave % TG, eg0 = wave / TG * NACC; // of a multiplying wavefront

    // Barrier s: stage s is in its tiles (and stage s - 3 is multiplied).  LDS writes only are
    // waited for: global loads stay in flight across it.
#define MOE_ROUTE_BARRIER()                                                                   \
    {                                                                                         \
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                                    \
        __builtin_amdgcn_s_barrier();                                                         \
        asm volatile("" ::: "memory");                                                        \
    }
    f32x4 acc[NACC];
    if (wave >= NC) {
        constexpr int VPT = RT::VPT, PD = RT::PD;
        const int ltid = tid - NC * 64;
        const char *src[VPT];
        int dst[VPT];
        bool is_x[VPT];
        int left[VPT];                                // columns of the row from the vector on, last stage
#pragma unroll
        for (int j = 0; j < VPT; ++j) {
            const int v = min(ltid + j * RT::NL * 64, RT::VECS - 1);    // (surplus repeats the last vector)
            is_x[j] = v < TB * RT::XV;
            if (is_x[j]) {
                const int row = v / RT::XV, vec = v % RT::XV;
                // bf16: eight consecutive columns, i.e. two steps; fp32: a lane's four of a quad
                const int col = sizeof(XT) == 2 ? vec * 8 : vec / 4 * 16 + vec % 4;
                src[j] = reinterpret_cast<const char *>(x + static_cast<size_t>(min(t0 + row, T - 1)) * d + col);
                left[j] = d - (nstage - 1) * kKC - col;
                dst[j] = row / 16 * TILE + col / 16 * QUAD + row % 16 * 16 +
                         (sizeof(XT) == 2 ? vec % 2 * 8 : vec % 4 * GROUP);
            } else {
                // (the packed matrix holds a lane's four columns of a quad side by side)
                const int row = (v - TB * RT::XV) / 16, q = v % 16 / 4, g = v % 4;
                src[j] = reinterpret_cast<const char *>(Wgp + static_cast<size_t>(min(row, EP - 1)) * dP + q * 16 + g * 4);
                left[j] = kKC;
                dst[j] = (TG + row / 16) * TILE + q * QUAD + g * GROUP + row % 16 * 16;
            }
        }
        u32x4 reg[PD][VPT];
        auto load = [&](auto slot, int s) {
#pragma unroll
            for (int j = 0; j < VPT; ++j) {
                u32x4 &q = reg[decltype(slot)::value][j];
                const char *p = src[j] + static_cast<size_t>(s) * (is_x[j] ? kKC * sizeof(XT) : kKC * 4);
                const int n = s == nstage - 1 ? left[j] : kKC;      // columns past d read as zeros
                q = (u32x4){0u, 0u, 0u, 0u};
                if (sizeof(XT) == 2 || !is_x[j]) {
                    if (n > 0) q = *reinterpret_cast<const u32x4 *>(p);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (n > 4 * i) q[i] = *reinterpret_cast<const uint32_t *>(p + 16 * i);
                }
            }
        };
        auto store = [&](auto slot, int at) {
#pragma unroll
            for (int j = 0; j < VPT; ++j) {
                char *o = tiles + at + dst[j];
                const u32x4 q = reg[decltype(slot)::value][j];
                if (sizeof(XT) == 2 && is_x[j]) {     // of every 16-lane group: its column of both steps
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        u32x2 p;
                        p[0] = g & 1 ? q[g >> 1] & 0xFFFF0000u : q[g >> 1] << 16;
                        p[1] = g & 1 ? q[2 + (g >> 1)] & 0xFFFF0000u : q[2 + (g >> 1)] << 16;
                        *reinterpret_cast<u32x2 *>(o + g * GROUP) = p;
                    }
                } else {
                    *reinterpret_cast<u32x4 *>(o) = q;
                }
            }
        };
        auto each = [&](auto body) {                  // body(0) .. body(PD - 1), compile-time
            body(std::integral_constant<int, 0>{});
            body(std::integral_constant<int, 1>{});
            if constexpr (PD > 2) body(std::integral_constant<int, 2>{});
            if constexpr (PD > 3) body(std::integral_constant<int, 3>{});
            if constexpr (PD > 4) body(std::integral_constant<int, 4>{});
            if constexpr (PD > 5) body(std::integral_constant<int, 5>{});
        };
        each([&](auto u) {
            if (decltype(u)::value < nstage) load(u, decltype(u)::value);
        });
        int at = 0;
        for (int s0 = 0; s0 < nstage; s0 += PD)
            each([&](auto u) {
                const int s = s0 + decltype(u)::value;
                if (s < nstage) {
                    store(u, at);
                    if (s + PD < nstage) load(u, s + PD);
                    MOE_ROUTE_BARRIER()
                    at = at == 2 * STAGE ? 0 : at + STAGE;
                }
            });
    } else {
#pragma unroll
        for (int a = 0; a < NACC; ++a) acc[a] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
        const char *const xlane = tiles + tg * TILE + kq * GROUP + r16 * 16;
        const char *const wlane = tiles + (TG + eg0) * TILE + kq * GROUP + r16 * 16;
        struct Quad {                                 // operands of four steps: 16 columns
            f32x4 x, w[NACC];
        } quad[4];
        auto read_part = [&](Quad &o, int at, int qd, int i) {
            if (i == 0) o.x = *reinterpret_cast<const f32x4 *>(xlane + at + qd * QUAD);
#pragma unroll
            for (int a = i; a < NACC; a += 4)
                o.w[a] = *reinterpret_cast<const f32x4 *>(wlane + at + a * TILE + qd * QUAD);
        };
        // multiplies one quad and issues the reads of the next but one between the steps; the
        // fences keep the compiler from moving them
        auto run_quad = [&](const Quad &use, Quad &fill, int fill_at, int fill_quad) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
#pragma unroll
                for (int a = 0; a < NACC; ++a)
                    acc[a] = __builtin_amdgcn_mfma_f32_16x16x4f32(use.w[a][i], use.x[i], acc[a], 0, 0, 0);
                read_part(fill, fill_at, fill_quad, i);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        MOE_ROUTE_BARRIER()
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            read_part(quad[0], 0, 0, i);
            read_part(quad[1], 0, 1, i);
        }
        // (behind the last stage the reads fetch a tile nobody multiplies)
        int at = 0;
        for (int s = 0; s < nstage; ++s) {
            const int next = at == 2 * STAGE ? 0 : at + STAGE;
            run_quad(quad[0], quad[2], at, 2);
            run_quad(quad[1], quad[3], at, 3);
            if (s + 1 < nstage) {
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            }
            run_quad(quad[2], quad[0], next, 0);
            run_quad(quad[3], quad[1], next, 1);
            at = next;
        }
    }
#undef MOE_ROUTE_BARRIER
    __syncthreads();                  // every wavefront is done with the tiles: reuse them for logits
    if (wave < NC) {
        const int xrow = tg * 16 + r16, t = t0 + xrow;
        // acc[a][r]: expert 16 (eg0 + a) + 4 kq + r, token r16 of the group
#pragma unroll
        for (int a = 0; a < NACC; ++a)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int e = (eg0 + a) * 16 + 4 * kq + r;
                if (e < E) {
                    float z = acc[a][r];
                    if (bias != nullptr && t < T) z = z + bias[static_cast<size_t>(t) * bias_stride + e];
                    zs[xrow][e] = z;
                }
            }
    }
    __syncthreads();
    // lanes per token in the tail, and logits per lane
    constexpr int LP = RT::NT / TB < EG * 16 ? RT::NT / TB : EG * 16, NQ = EG * 16 / LP;
    tail.template run<NQ, LP, TB>(zs, t0, T, E);
}

// Gate matrix [d][E] (fp32 or bf16) -> fp32 [EP][dP], expert-major, zero padded, each run of 16
// columns in the order packed_gate_column gives.
template <typename XT>
__global__ void pack_gate_kernel(const XT *__restrict__ Wg, float *__restrict__ Wgp,
                                 int d, int dP, int E, int EP)
{
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= dP * EP) return;
    const int e = idx / dP, i = packed_gate_column(idx % dP);
    float v = 0.0f;
    if (e < E && i < d) {
        if constexpr (sizeof(XT) == 2)
            v = bf16_to_f32(Wg[static_cast<size_t>(i) * E + e]);
        else
            v = Wg[static_cast<size_t>(i) * E + e];
    }
    Wgp[idx] = v;
}

int pow2_ceil(int v)
{
    int p = 1;
    while (p < v) p <<= 1;
    return p;
}

int padded_dim(int d) { return (d + kGatePad - 1) / kGatePad * kGatePad; }

// Tokens per block (= per segment of the dispatch plan): 16, the least the matrix instruction
// takes, as long as the plan stays within the 512 segments that one launch ranks; more where
// that many blocks would only read the gate matrix more often.
int route_tokens(const moe_shape &s) { return s.T <= 16 * 512 ? 16 : s.T <= 32 * 512 ? 32 : 64; }

// tokens: of the T of the shape (which choose the tile), those of this launch
template <typename XT, typename Tail>
moe_status launch_route_t(const moe_shape &s, int tokens, const XT *x, const float *Wgp,
                          const float *bias, int bias_stride, const Tail &tail, hipStream_t st)
{
    const int EP = pow2_ceil(s.E);
    const int dP = padded_dim(s.d_model);
    const int tb = route_tokens(s), eg = EP <= 16 ? 1 : EP / 16;
    bool launched = false;
#define MOE_ROUTE_CASE(TB_, EG_)                                                              \
    if (tb == TB_ && eg == EG_) {                                                             \
        auto kern = route_mfma_kernel<XT, TB_, EG_, Tail>;                                       \
        constexpr size_t lds = RouteTile<XT, TB_, EG_>::LDS;                                  \
        static PerDeviceOnce once;                                                            \
        once.raise_lds(reinterpret_cast<const void *>(kern), static_cast<int>(lds));          \
        hipLaunchKernelGGL(kern, dim3(ceil_div(tokens, TB_)), dim3(RouteTile<XT, TB_, EG_>::NT), lds, st, x,  \
                           Wgp, bias, bias_stride, tail, tokens, s.d_model, dP, s.E, EP);     \
        launched = true;                                                                      \
    }
    MOE_ROUTE_CASE(16, 1) MOE_ROUTE_CASE(16, 2) MOE_ROUTE_CASE(16, 4)
    MOE_ROUTE_CASE(32, 1) MOE_ROUTE_CASE(32, 2) MOE_ROUTE_CASE(32, 4)
    MOE_ROUTE_CASE(64, 1) MOE_ROUTE_CASE(64, 2) MOE_ROUTE_CASE(64, 4)
#undef MOE_ROUTE_CASE
    if (!launched) {
        set_error("route: internal error, %d tokens x %d experts", tb, EP);
        return MOE_EINVAL;
    }
    MOE_TRY_HIP(hipGetLastError());
    return MOE_OK;
}

}  // namespace

int route_segment_tokens(const moe_shape &s) { return route_tokens(s); }

size_t packed_gate_bytes(const moe_shape &s)
{
    return static_cast<size_t>(padded_dim(s.d_model)) * pow2_ceil(s.E) * sizeof(float);
}

moe_status launch_pack_gate(const moe_shape &s, const void *Wg, float *Wgp, hipStream_t st)
{
    const int EP = pow2_ceil(s.E);
    const int dP = padded_dim(s.d_model);
    const int n = dP * EP;
    const dim3 grid(ceil_div(n, 256)), block(256);
    if (s.dtype == MOE_BF16)
        hipLaunchKernelGGL(pack_gate_kernel<uint16_t>, grid, block, 0, st,
                           static_cast<const uint16_t *>(Wg), Wgp, s.d_model, dP, s.E, EP);
    else
        hipLaunchKernelGGL(pack_gate_kernel<float>, grid, block, 0, st,
                           static_cast<const float *>(Wg), Wgp, s.d_model, dP, s.E, EP);
    MOE_TRY_HIP(hipGetLastError());
    return MOE_OK;
}

moe_status launch_route(const moe_shape &s, const void *x, const void *Wgp,
                        const float *bias, int bias_stride, int32_t *expert_idx,
                        float *gate, int32_t *seg_cnt, hipStream_t st)
{
    const RouteTail tail{expert_idx, gate, seg_cnt, s.k, s.renorm_topk};
    if (s.dtype == MOE_BF16)
        return launch_route_t(s, s.T, static_cast<const uint16_t *>(x), static_cast<const float *>(Wgp),
                              bias, bias_stride, tail, st);
    return launch_route_t(s, s.T, static_cast<const float *>(x), static_cast<const float *>(Wgp), bias,
                          bias_stride, tail, st);
}

// The logit gradients of tokens [t0, t1) of a bf16 layer: dz [T][E] from dgate [T][k].  The logits
// are computed again, the same chain as in the forward pass.
moe_status launch_gate_grad(const moe_shape &s, int t0, int t1, const uint16_t *x, const float *Wgp,
                            const float *bias, int bias_stride, const int32_t *expert_idx,
                            const float *dgate, float *dz, hipStream_t st)
{
    const size_t t = static_cast<size_t>(t0);
    const GateGradTail tail{expert_idx + t * s.k, dgate + t * s.k, dz + t * s.E, s.k};
    return launch_route_t(s, t1 - t0, x + t * s.d_model, Wgp, bias != nullptr ? bias + t * bias_stride : nullptr,
                          bias_stride, tail, st);
}

}  // namespace moe
