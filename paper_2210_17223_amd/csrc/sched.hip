// Popularity-based expert scheduling for inference (paper Sec. 5.2): sample-path tables,
// the per-batch popularity estimate in exact fixed-point arithmetic, Eq. (1),
// first-fit-decreasing packing and the two-phase check.  The table and estimate steps
// are integer kernels over tokens (HBM / atomic bound, a few bytes per token); the
// scheduling decisions are tiny and run on the host thread that owns the scheduler.
#include "common.h"
#include "moe_sched.h"

#include <algorithm>

namespace moe {
namespace {

constexpr int kFix = 32;           // probabilities are floor(p * 2^32)
constexpr int64_t kMaxPaths = 1ll << 24;

int64_t path_count(const moe_path_shape *s)
{
    if (s == nullptr || s->E < 1 || s->E > kMaxExperts || s->l < 1 || s->k < 1 ||
        s->k > kMaxTopK || s->k > s->E)
        return 0;
    int64_t p = 1;
    for (int m = 0; m < s->l; ++m) {
        p *= s->E;
        if (p > kMaxPaths) return 0;
    }
    return p;
}

// Sample path of token t whose oldest layer starts at `hist` (layer stride = T*k entries):
// the l first choices as an l-digit number in base E, or -1 if one is not an expert.
__device__ __forceinline__ int path_of(const int32_t *__restrict__ hist, size_t layer_stride,
                                       int t, int k, int l, int E)
{
    int j = 0;
    for (int m = 0; m < l; ++m) {
        const int e = hist[m * layer_stride + static_cast<size_t>(t) * k];
        if (static_cast<unsigned>(e) >= static_cast<unsigned>(E)) return -1;
        j = j * E + e;
    }
    return j;
}

// Work-items of a launch are counted in 32 bits, and the runtime drops what is above them without an
// error: kernels whose work may be more walk it with at most so many blocks of 256.
constexpr int64_t kMostBlocks = 1 << 20;

// One thread per (table a, token t): table a predicts layer a + l from layers a .. a+l-1.
__global__ __launch_bounds__(256) void path_profile_kernel(
    const int32_t *__restrict__ sel, uint32_t *__restrict__ counts, int T, int tables, int E,
    int k, int l, int paths)
{
    const long n = static_cast<long>(tables) * T, step = static_cast<long>(gridDim.x) * blockDim.x;
    for (long idx = static_cast<long>(blockIdx.x) * blockDim.x + threadIdx.x; idx < n; idx += step) {
        const int a = static_cast<int>(idx / T), t = static_cast<int>(idx % T);
        const size_t layer_stride = static_cast<size_t>(T) * k;
        const int j = path_of(sel + a * layer_stride, layer_stride, t, k, l, E);
        bool valid = j >= 0;
        const int32_t *next = sel + (a + l) * layer_stride + static_cast<size_t>(t) * k;
        for (int c = 0; c < k; ++c) valid = valid && static_cast<unsigned>(next[c]) < static_cast<unsigned>(E);
        if (!valid) continue;
        uint32_t *row = counts + (static_cast<size_t>(a) * paths + j) * E;
        for (int c = 0; c < k; ++c) atomicAdd(&row[next[c]], 1u);
    }
}

// The same counts for batches of many tokens.  Popular experts put a large share of the tokens
// on a few counters, and the global atomics on those serialise; here a block counts its share of one
// table's tokens in LDS and adds what it counted to the table, one global atomic per counter.
//   DIRECT: the table's counters as 16-bit halves of LDS words (a share adds at most 65535 to any).
//   else:   LDS is a hash table of 2^slot_bits (counter, count) pairs, first come first served: the
//           popular counters are there early, a counter that finds its two places taken goes to
//           global memory.
// LL: l where it is 2 or 3, else 0: with l known all l + 1 choices of four tokens are on their way at
// once, and a block waits once a round for them instead of l + 4 times.
// Bound by reading the choices (9 of 45 us below) and by the flush (18: its atomics; two neighbouring
// counters go in one 64-bit add, whose low half does not overflow because row totals stay below
// 2^32).  2^20 tokens, 12 layers, 16 experts, paths of length 3: 45 us (75 with one wait per choice and
// 32-bit adds, 5050 with a global atomic per token and table); k = 2 70 (121).  Tables past LDS: bound
// by their scattered atomics, fewer of them the more tokens share a hash table: 32 experts, 6 layers, 2^20
// tokens 96 us (128 with 2^13 places and two blocks per unit), k = 2 193 (276; 255 before the waits went);
// uniform choices, which share no counters, 124 either way.
constexpr int kProfThreads = 1024;
constexpr int kMostSlotBits = 14;                          // one block per compute unit
constexpr int kProfMinTokens = 4096;                       // fewer: not worth clearing and flushing LDS
constexpr int kProfLdsCounters = 73728;                    // 144 KiB of 16-bit counters

template <bool DIRECT, int LL>
__global__ __launch_bounds__(kProfThreads) void path_profile_lds_kernel(
    const int32_t *__restrict__ sel, uint32_t *__restrict__ counts, int T, int share, int splits,
    int E, int k, int l, int paths, int slot_bits)
{
    const int slots = 1 << slot_bits;
    constexpr uint32_t kEmpty = 0xFFFFFFFFu;
    extern __shared__ uint32_t lds[];
    const int tid = threadIdx.x;
    const int a = blockIdx.x / splits;
    const long t0 = static_cast<long>(blockIdx.x % splits) * share;
    const int t1 = static_cast<int>(min(t0 + share, static_cast<long>(T)));
    const size_t n = static_cast<size_t>(paths) * E, layer_stride = static_cast<size_t>(T) * k;
    const int words = DIRECT ? static_cast<int>((n + 1) / 2) : 2 * slots;
    for (int i = tid; i < words; i += kProfThreads) lds[i] = DIRECT || i >= slots ? 0u : kEmpty;
    __syncthreads();

    const int32_t *hist = sel + a * layer_stride;
    const int32_t *next = sel + (a + l) * layer_stride;
    uint32_t *table = counts + static_cast<size_t>(a) * n;
    auto count = [&](uint32_t key) {
        if constexpr (DIRECT) {
            atomicAdd(&lds[key >> 1], 1u << (16 * (key & 1u)));
        } else {
            uint32_t at = (key * 2654435761u) >> (32 - slot_bits);
            for (int probe = 0; probe < 2; ++probe, at ^= 1u) {
                uint32_t have = *static_cast<volatile uint32_t *>(&lds[at]);
                if (have == kEmpty) have = atomicCAS(&lds[at], kEmpty, key);
                if (have == kEmpty || have == key) {
                    atomicAdd(&lds[slots + at], 1u);
                    return;
                }
            }
            atomicAdd(&table[key], 1u);
        }
    };
    // four tokens per thread at a time: their loads are in flight together
    constexpr int U = 4;
    const int second = min(1, k - 1);
    for (long tb = t0 + tid; tb < t1; tb += U * kProfThreads) {
        int j[U], first_next[U], second_next[U];
        size_t at[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            j[u] = 0;
            ok[u] = tb + u * kProfThreads < t1;
            at[u] = static_cast<size_t>(min(tb + u * kProfThreads, static_cast<long>(t1) - 1)) * k;
            first_next[u] = next[at[u]];
            second_next[u] = next[at[u] + second];
        }
        auto extend = [&](const int (&e)[U]) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                ok[u] = ok[u] && static_cast<unsigned>(e[u]) < static_cast<unsigned>(E);
                j[u] = ok[u] ? j[u] * E + e[u] : 0;
            }
        };
        if constexpr (LL != 0) {
            int e[LL][U];
#pragma unroll
            for (int m = 0; m < LL; ++m)
#pragma unroll
                for (int u = 0; u < U; ++u) e[m][u] = hist[m * layer_stride + at[u]];
#pragma unroll
            for (int m = 0; m < LL; ++m) extend(e[m]);
        } else {
            for (int m = 0; m < l; ++m) {
                int e[U];
#pragma unroll
                for (int u = 0; u < U; ++u) e[u] = hist[m * layer_stride + at[u]];
                extend(e);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            bool valid = ok[u] && static_cast<unsigned>(first_next[u]) < static_cast<unsigned>(E) &&
                         static_cast<unsigned>(second_next[u]) < static_cast<unsigned>(E);
            if (!valid) continue;
            const int32_t *choice = next + at[u];
            for (int c = 2; c < k; ++c) valid = valid && static_cast<unsigned>(choice[c]) < static_cast<unsigned>(E);
            if (!valid) continue;
            const uint32_t row = static_cast<uint32_t>(j[u]) * E;
            count(row + first_next[u]);
            if (k > 1) count(row + second_next[u]);
            for (int c = 2; c < k; ++c) count(row + choice[c]);
        }
    }
    __syncthreads();
    if constexpr (DIRECT) {
        if (n % 2 == 0 && reinterpret_cast<uintptr_t>(table) % 8 == 0) {
            unsigned long long *pairs = reinterpret_cast<unsigned long long *>(table);
            for (int i = tid; i < words; i += kProfThreads) {
                const unsigned long long v = lds[i];
                if (v != 0) atomicAdd(&pairs[i], (v & 0xFFFFu) | (v >> 16 << 32));
            }
            return;
        }
        for (int i = tid; i < words; i += kProfThreads) {
            const uint32_t v = lds[i];
            if (v & 0xFFFFu) atomicAdd(&table[2 * i], v & 0xFFFFu);
            if (v >> 16) atomicAdd(&table[2 * i + 1], v >> 16);
        }
    } else {
        for (int i = tid; i < slots; i += kProfThreads)
            if (lds[slots + i] != 0u) atomicAdd(&table[lds[i]], lds[slots + i]);
    }
}

// Sixteen lanes per (table, path) row, up to four counters each: row total, then k rounds of
// "largest remaining count, lowest index first" as a maximum over the lanes.  (36864
// rows of 16: 5.2 us; 6.0 with one thread per row reading it k + 1 times.)
__global__ __launch_bounds__(256) void path_finalize_kernel(
    const uint32_t *__restrict__ counts, int32_t *__restrict__ top_expert,
    unsigned long long *__restrict__ top_prob, long rows, int E, int k)
{
    constexpr int LP = 16, NQ = kMaxExperts / LP;
    const long step = static_cast<long>(gridDim.x) * (blockDim.x / LP);
    const int sub = threadIdx.x % LP;
    // (whole groups of sixteen lanes leave the loop together)
    for (long r = static_cast<long>(blockIdx.x) * (blockDim.x / LP) + threadIdx.x / LP; r < rows; r += step) {
        const uint32_t *row = counts + r * E;
        uint32_t v[NQ];
        unsigned long long tot = 0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int e = sub + LP * q;
            v[q] = e < E ? row[e] : 0u;
            tot += v[q];
        }
#pragma unroll
        for (int m = 1; m < LP; m <<= 1) tot += __shfl_xor(tot, m);
        for (int c = 0; c < k; ++c) {
            unsigned long long best = 0;               // count, then 63 - index; count 0 never wins
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const unsigned long long key = static_cast<unsigned long long>(v[q]) << 6 | (63 - sub - LP * q);
                if (v[q] != 0u && key > best) best = key;
            }
#pragma unroll
            for (int m = 1; m < LP; m <<= 1) best = max(best, __shfl_xor(best, m));
            const int e = best != 0 ? 63 - static_cast<int>(best & 63u) : -1;
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                if (e == sub + LP * q) v[q] = 0u;
            if (sub == 0) {
                top_expert[r * k + c] = e;
                top_prob[r * k + c] = e >= 0 ? ((best >> 6) << kFix) / tot : 0ull;
            }
        }
    }
}

__global__ void zero_u64_kernel(unsigned long long *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// A block walks its share of the tokens, sums their contributions in LDS and adds them to
// S with one 64-bit atomic per expert (few blocks: the atomics of all blocks hit the same E
// addresses).  Integer sums: the result does not depend on the order.
__global__ __launch_bounds__(256) void popularity_estimate_kernel(
    const int32_t *__restrict__ hist, const int32_t *__restrict__ top_expert,
    const unsigned long long *__restrict__ top_prob, unsigned long long *__restrict__ S,
    int N_t, int E, int k, int l)
{
    __shared__ unsigned long long acc[kMaxExperts];
    if (threadIdx.x < kMaxExperts) acc[threadIdx.x] = 0ull;
    __syncthreads();
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < N_t; t += gridDim.x * blockDim.x) {
        const int j = path_of(hist, static_cast<size_t>(N_t) * k, t, k, l, E);
        if (j < 0) continue;
        for (int c = 0; c < k; ++c) {
            const int e = top_expert[static_cast<size_t>(j) * k + c];
            if (e >= 0) atomicAdd(&acc[e], top_prob[static_cast<size_t>(j) * k + c]);
        }
    }
    __syncthreads();
    if (static_cast<int>(threadIdx.x) < E && acc[threadIdx.x] != 0ull) atomicAdd(&S[threadIdx.x], acc[threadIdx.x]);
}

bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// The packing of moe_schedule_experts, straight into the caller's arrays (at most kMaxExperts experts:
// nothing is allocated).
void schedule_experts(int N, int E, const uint64_t *w, uint64_t W, const uint8_t *has, int max_pack,
                      int32_t *replicas, int32_t *dev_count, int32_t *dev_experts, int32_t *devices_used)
{
    std::fill(replicas, replicas + E, 0);
    std::fill(dev_count, dev_count + N, 0);
    std::fill(dev_experts, dev_experts + static_cast<size_t>(N) * E, -1);
    // wrapping can bring an expert to a device that hosts it already: never more than E per device
    auto host = [&](int64_t d, int32_t e) {
        int32_t *list = dev_experts + d * E;
        if (std::find(list, list + dev_count[d], e) == list + dev_count[d]) list[dev_count[d]++] = e;
    };
    int64_t used = 0;                             // devices asked for
    int small[kMaxExperts], n_small = 0;          // heaviest first, index order kept on ties
    for (int e = 0; e < E; ++e) {
        if (!has[e]) continue;
        if (w[e] >= W) {
            // round half up of w / W, without forming 2w + W (which could overflow)
            const uint64_t q = w[e] / W, rem = w[e] % W;
            const uint64_t r = q + (rem >= W - rem ? 1 : 0);
            replicas[e] = static_cast<int32_t>(std::min<uint64_t>(r, N));   // never more than all devices
            for (int32_t i = 0; i < replicas[e]; ++i) host(used++ % N, e);
        } else {
            int at = n_small++;
            for (; at > 0 && w[small[at - 1]] < w[e]; --at) small[at] = small[at - 1];
            small[at] = e;
        }
    }
    int n_bins = 0, in_bin[kMaxExperts], bin_of[kMaxExperts];
    uint64_t load[kMaxExperts];
    for (int i = 0; i < n_small; ++i) {
        const int e = small[i];
        int b = 0;
        while (b < n_bins && !(load[b] + w[e] <= W && in_bin[b] < max_pack)) ++b;
        if (b == n_bins) load[n_bins] = 0, in_bin[n_bins] = 0, ++n_bins;
        bin_of[i] = b;
        load[b] += w[e];
        ++in_bin[b];
        replicas[e] = 1;
    }
    for (int b = 0; b < n_bins; ++b, ++used)
        for (int i = 0; i < n_small; ++i)
            if (bin_of[i] == b) host(used % N, small[i]);
    const int64_t free_devs = N - used;
    int64_t m = 0;
    for (int e = 0; e < E; ++e) {
        if (has[e]) continue;
        host(free_devs > 0 ? used + m % free_devs : e % N, e);
        replicas[e] = 1;
        ++m;
    }
    *devices_used = static_cast<int32_t>(std::min<int64_t>(used, N));
}

moe_status check_schedule_args(int32_t N, int32_t E, const void *w_or_S, int32_t max_pack,
                               const int32_t *replicas, const int32_t *dev_count,
                               const int32_t *dev_experts, const int32_t *devices_used)
{
    if (N < 1 || E < 1 || E > kMaxExperts || max_pack < 1) {
        set_error("schedule: need N >= 1, 1 <= E <= %d, max_pack >= 1 (N=%d E=%d max_pack=%d)",
                  kMaxExperts, N, E, max_pack);
        return MOE_EINVAL;
    }
    if (w_or_S == nullptr || replicas == nullptr || dev_count == nullptr ||
        dev_experts == nullptr || devices_used == nullptr) {
        set_error("schedule: NULL argument");
        return MOE_EINVAL;
    }
    return MOE_OK;
}

// The m most popular experts, most popular first, ties to the lower index.
template <typename V>
void top_list(int E, int m, const V *score, int *order)
{
    int n = 0;
    for (int e = 0; e < E; ++e) {
        int at = n;
        for (; at > 0 && score[order[at - 1]] < score[e]; --at)
            if (at < m) order[at] = order[at - 1];
        if (at < m) order[at] = e;
        n = std::min(n + 1, m);
    }
}

}  // namespace
}  // namespace moe

using namespace moe;

extern "C" {

int64_t moe_path_count(const moe_path_shape *s) { return path_count(s); }

moe_status moe_path_profile(const moe_path_shape *s, const int32_t *sel, int32_t T,
                            uint32_t *counts, void *stream)
{
    const int64_t paths = path_count(s);
    if (paths == 0 || s->L <= s->l) {
        set_error("path shape: need 1 <= E <= %d, 1 <= k <= min(E, %d), l >= 1, E^l <= 2^24, L > l",
                  kMaxExperts, kMaxTopK);
        return MOE_EINVAL;
    }
    if (T < 0 || sel == nullptr || counts == nullptr || !aligned(sel, 4) || !aligned(counts, 4)) {
        set_error("moe_path_profile: T < 0, or sel / counts NULL or misaligned");
        return MOE_EINVAL;
    }
    const int tables = s->L - s->l;
    const long n = static_cast<long>(tables) * T;
    if (n == 0) return MOE_OK;
    if (n > (1l << 40)) {
        set_error("moe_path_profile: %ld (table, token) pairs in one call", n);
        return MOE_EUNSUPPORTED;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t counters = paths * s->E;
    if (T < kProfMinTokens) {
        const int64_t blocks = std::min<int64_t>((n + 255) / 256, kMostBlocks);
        hipLaunchKernelGGL(path_profile_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, sel, counts, T, tables, s->E, s->k,
                           s->l, static_cast<int>(paths));
    } else {
        const bool direct = counters <= kProfLdsCounters;
        size_t lds = direct ? align_up(static_cast<size_t>(counters) * 2, 4) : size_t(8) << kMostSlotBits;
        // shares: one block per compute unit (two where the LDS of both fits), or as many times
        // that as keep a share's counts below 2^16
        const int per_cu = lds <= 64 * 1024 ? 2 : 1;
        int64_t splits = std::max(1, 256 * per_cu / tables);
        const int64_t most = 65535 / s->k, least = (T + most - 1) / most;
        splits *= (least + splits - 1) / splits;
        splits = std::min<int64_t>(splits, (T + kProfThreads - 1) / kProfThreads);
        const int64_t share = (T + splits - 1) / splits;
        // A block of at most one token per thread, as few tokens make them, meets fewer counters than it takes to
        // clear and flush the larger table: us with 2^13 / 2^14 places, 32 experts, 6 layers, l = 3: 16384
        // tokens, k = 2 11.5 / 12.2, 65536 tokens, k = 1 16.0 / 16.6 (uniform choices 12.1 / 12.9); with
        // larger shares (and twice the blocks for 2^13) 90000 23.0 / 20.9, 131072 36.3 / 25.0 (uniform choices
        // 18.5 / 15.5, 21.4 / 20.4).
        const int slot_bits = share <= kProfThreads ? kMostSlotBits - 1 : kMostSlotBits;
        if (!direct) lds = size_t(8) << slot_bits;
        if (tables * splits >= (1ll << 32) / kProfThreads) {
            set_error("moe_path_profile: %d tables of %d tokens in one call", tables, T);
            return MOE_EUNSUPPORTED;
        }
        auto kern = s->l == 2   ? direct ? path_profile_lds_kernel<true, 2> : path_profile_lds_kernel<false, 2>
                    : s->l == 3 ? direct ? path_profile_lds_kernel<true, 3> : path_profile_lds_kernel<false, 3>
                    : direct    ? path_profile_lds_kernel<true, 0> : path_profile_lds_kernel<false, 0>;
        static PerDeviceOnce once[3][2];
        once[s->l == 2 ? 1 : s->l == 3 ? 2 : 0][direct].raise_lds(reinterpret_cast<const void *>(kern), direct ? kProfLdsCounters * 2 : 8 << kMostSlotBits);
        hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(tables * splits)), dim3(kProfThreads), lds, st,
                           sel, counts, T, static_cast<int>(share), static_cast<int>(splits), s->E,
                           s->k, s->l, static_cast<int>(paths), slot_bits);
    }
    MOE_TRY_HIP(hipGetLastError());
    return MOE_OK;
}

moe_status moe_path_finalize(const moe_path_shape *s, const uint32_t *counts,
                             int32_t *top_expert, uint64_t *top_prob, void *stream)
{
    const int64_t paths = path_count(s);
    if (paths == 0 || s->L <= s->l) {
        set_error("path shape: need 1 <= E <= %d, 1 <= k <= min(E, %d), l >= 1, E^l <= 2^24, L > l",
                  kMaxExperts, kMaxTopK);
        return MOE_EINVAL;
    }
    if (counts == nullptr || top_expert == nullptr || top_prob == nullptr || !aligned(counts, 4) ||
        !aligned(top_expert, 4) || !aligned(top_prob, 8)) {
        set_error("moe_path_finalize: NULL or misaligned argument");
        return MOE_EINVAL;
    }
    const long rows = static_cast<long>(s->L - s->l) * paths;
    const int64_t blocks = std::min<int64_t>((rows + 15) / 16, kMostBlocks);
    hipLaunchKernelGGL(path_finalize_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), counts, top_expert,
                       reinterpret_cast<unsigned long long *>(top_prob), rows, s->E, s->k);
    MOE_TRY_HIP(hipGetLastError());
    return MOE_OK;
}

moe_status moe_popularity_estimate(const moe_path_shape *s, const int32_t *sel_hist,
                                   int32_t N_t, const int32_t *top_expert,
                                   const uint64_t *top_prob, uint64_t *S, void *stream)
{
    if (path_count(s) == 0) {
        set_error("path shape: need 1 <= E <= %d, 1 <= k <= min(E, %d), l >= 1, E^l <= 2^24",
                  kMaxExperts, kMaxTopK);
        return MOE_EINVAL;
    }
    if (N_t < 0 || sel_hist == nullptr || top_expert == nullptr || top_prob == nullptr ||
        S == nullptr || !aligned(sel_hist, 4) || !aligned(top_expert, 4) ||
        !aligned(top_prob, 8) || !aligned(S, 8)) {
        set_error("moe_popularity_estimate: N_t < 0, or a NULL or misaligned argument");
        return MOE_EINVAL;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    unsigned long long *Sd = reinterpret_cast<unsigned long long *>(S);
    hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(kMaxExperts), 0, st, Sd, s->E);
    if (N_t > 0)
        hipLaunchKernelGGL(popularity_estimate_kernel,
                           dim3(std::min(256, (N_t + 1023) / 1024)), dim3(256), 0, st,
                           sel_hist, top_expert,
                           reinterpret_cast<const unsigned long long *>(top_prob), Sd, N_t, s->E,
                           s->k, s->l);
    MOE_TRY_HIP(hipGetLastError());
    return MOE_OK;
}

double moe_devices_for_expert(uint64_t S_e, int32_t N_t, int32_t N)
{
    if (N_t < 1) return 0.0;
    return static_cast<double>(N) * (static_cast<double>(S_e) / 4294967296.0) /
           static_cast<double>(N_t);
}

moe_status moe_schedule_experts(int32_t N, int32_t E, const uint64_t *w, uint64_t W,
                                const uint8_t *has, int32_t max_pack, int32_t *replicas,
                                int32_t *dev_count, int32_t *dev_experts, int32_t *devices_used)
{
    const moe_status st =
        check_schedule_args(N, E, w, max_pack, replicas, dev_count, dev_experts, devices_used);
    if (st != MOE_OK) return st;
    if (has == nullptr || W < 1) {
        set_error("moe_schedule_experts: has is NULL or W < 1");
        return MOE_EINVAL;
    }
    schedule_experts(N, E, w, W, has, max_pack, replicas, dev_count, dev_experts, devices_used);
    return MOE_OK;
}

int32_t moe_top_lists_identical(int32_t E, int32_t k, const uint64_t *S, const int32_t *counts)
{
    if (E < 1 || E > kMaxExperts || k < 1 || S == nullptr || counts == nullptr) return 0;
    const int m = k > E / 2 ? E : 2 * k;
    int by_estimate[kMaxExperts], by_count[kMaxExperts];
    top_list(E, m, S, by_estimate);
    top_list(E, m, counts, by_count);
    return std::equal(by_estimate, by_estimate + m, by_count) ? 1 : 0;
}

moe_status moe_schedule_layer(int32_t N, int32_t E, int32_t k, int32_t N_t, const uint64_t *S,
                              const int32_t *counts, int32_t max_pack, int32_t *replicas,
                              int32_t *dev_count, int32_t *dev_experts, int32_t *devices_used,
                              int32_t *rescheduled)
{
    const moe_status st =
        check_schedule_args(N, E, S, max_pack, replicas, dev_count, dev_experts, devices_used);
    if (st != MOE_OK) return st;
    if (counts == nullptr || rescheduled == nullptr || k < 1 || N_t < 1) {
        set_error("moe_schedule_layer: counts / rescheduled NULL, or k < 1, or N_t < 1");
        return MOE_EINVAL;
    }
    // N * S[e] <= N * N_t * 2^32 must fit 64 bits
    if (static_cast<uint64_t>(N) * static_cast<uint64_t>(N_t) >= (1ull << 31)) {
        set_error("moe_schedule_layer: N * N_t = %llu does not fit the fixed-point weights",
                  static_cast<unsigned long long>(N) * static_cast<unsigned long long>(N_t));
        return MOE_EUNSUPPORTED;
    }
    uint64_t w[kMaxExperts];
    uint8_t has[kMaxExperts];
    *rescheduled = 0;
    if (moe_top_lists_identical(E, k, S, counts)) {
        for (int e = 0; e < E; ++e) {
            w[e] = static_cast<uint64_t>(N) * S[e];
            has[e] = S[e] > 0;
        }
        schedule_experts(N, E, w, static_cast<uint64_t>(N_t) << kFix, has, max_pack, replicas, dev_count,
                         dev_experts, devices_used);
    } else {
        for (int e = 0; e < E; ++e) {
            w[e] = static_cast<uint64_t>(N) * static_cast<uint64_t>(counts[e] < 0 ? 0 : counts[e]);
            has[e] = counts[e] > 0;
        }
        schedule_experts(N, E, w, static_cast<uint64_t>(N_t) * k, has, max_pack, replicas, dev_count,
                         dev_experts, devices_used);
        *rescheduled = 1;
    }
    return MOE_OK;
}

}  // extern "C"
