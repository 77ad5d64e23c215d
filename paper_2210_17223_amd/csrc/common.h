// Shared declarations of libmoe's translation units (host helpers, device
// conversions, kernel launch prototypes).  gfx950 only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <mutex>

#include "moe.h"

namespace moe {

constexpr int kWave = 64;          // wavefront width on CDNA
constexpr int kMaxExperts = 64;    // one ballot bit / one lane per expert
constexpr int kMaxTopK = 8;
constexpr int kSegTok = 64;        // most tokens per plan segment (= tokens per gate block)
constexpr int kMaxChunks = 64;

// ---- host side -------------------------------------------------------------
void set_error(const char *fmt, ...);
moe_status hip_fail(hipError_t e, const char *what);

#define MOE_TRY_HIP(expr)                                             \
    do {                                                              \
        hipError_t e_ = (expr);                                       \
        if (e_ != hipSuccess) return ::moe::hip_fail(e_, #expr);      \
    } while (0)

// Raises a kernel's dynamic-LDS limit once per kernel and per device.  Any host thread may be
// the first to launch a kernel: the flag word is atomic, and a thread that arrives while
// another is still setting the attribute waits for it instead of launching too early.
struct PerDeviceOnce {
    std::atomic<uint64_t> done{0};           // bit per device ordinal (up to 64 devices)
    std::mutex setting;
    void raise_lds(const void *kernel, int bytes)
    {
        int dev = 0;
        (void)hipGetDevice(&dev);
        const uint64_t bit = 1ull << (dev & 63);
        if (done.load(std::memory_order_acquire) & bit) return;
        std::lock_guard<std::mutex> lock(setting);
        if (done.load(std::memory_order_relaxed) & bit) return;
        (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        done.fetch_or(bit, std::memory_order_release);
    }
};

__host__ __device__ inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
__host__ __device__ inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// One output tile of a grouped GEMM: rows [row0, row1) of the expert-major buffer, all
// owned by `expert`, output columns [n0, n0 + tile width).  expert < 0: no tile.
struct WorkItem {
    int32_t expert;
    int32_t row0;
    int32_t row1;
    int32_t n0;
};

// Tile shape and work-list bounds of one of the two expert GEMMs.
struct GemmPlan {
    int32_t bm, bn;          // rows / columns per output tile; bm: the most rows of a work item
    bool w4 = false;         // the four-wavefront kernels (gemm_w4.h)
    bool deep = false;       // 128 x 128, one block per compute unit with five stages on their way
    int32_t tiles_n;         // column tiles
    int32_t max_row_tiles;   // upper bound of row tiles per list
    int32_t max_items;       // entries of a work list (a multiple of 8; surplus ones hold no tile)
    int32_t concurrent;      // work items in flight per XCD (sets the panel width)
};
// Entries of a work list: a block each, and a multiple of the eight L2s the blocks go round.
inline int32_t work_list_entries(const GemmPlan &gp) { return (gp.max_row_tiles * gp.tiles_n + 7) / 8 * 8; }
// Tile of a row-grouped GEMM on the four-wavefront kernels (gemm_w4.h): `rows` rows in all over E
// experts.  256 x 256 where there are many such tiles, unless the contraction is one of a few
// stages that 128 x 128 tiles hide their prologue and epilogue behind better.  The larger tile's time over
// the smaller's, 4800 forward GEMMs of 8000 .. 130000 rows: 1.05 at K = 512, 1.03 at 640, 0.99 at 768, 0.97 at 896,
// 0.96 at 1024, 0.88 at 1600 .. 2047; but the product that dP is made of, over 130 layers, 1.26 at 704 .. 895 and 1.17
// at 896 .. 1023, hence 1024 for both.  Below four stages the larger tile takes 1.34 / 1.29 / 1.23 times as long at
// K = 64 / 128 / 192 and stays: the tests of a loop that ends before it is under way run there.
// Where tiles are few, by the number of rounds the tiles take on the chip -- 256 of 256 x 256 at a
// time, 512 of 128 x 128 (two per compute unit), and a tile's time in 64-deep stages -- with the
// times measured over layers of 256 .. 20000 tokens (us: a 256 x 256 stage 1.25, or 1.5 once the
// chip is full and lowers its clock, prologue and epilogue 10; a round of 128 x 128 0.85, or 0.55
// where compute units hold one, and 3; rows that do not start on 128-byte lines cost the smaller
// tile 1.7 times as much).  E.g. rows, E, N, K -> us of the layer with 256 x 256 / 128 x 128:
// 24249, 8, 1152, 2560 344 / 384; 12092, 8, 1024, 2624 182 / 189; 6002, 13, 1000, 2600 176 / 195;
// 23127, 64, 1600, 512 202 / 173; 8192, 16, 768, 3072 150 / 130; 39780, 16, 7048, 2032 2674 / 3003.
// 128 x 256 instead of 128 x 128 for long contractions with more tiles than the chip takes one per
// unit of.  Its time over the smaller tile's on that side of the line: 0.93 over 760 GEMMs whose last column
// tile is more than half full, 1.04 over 680 others when rows spread evenly; over 470 layers of uneven and even rows
// of the latter kind the smaller tile would cost 1.01 (second GEMM), 1.02 (dxe) and 1.04 (first GEMM of a stack).  On the other
// side: K = 1024 .. 1535 1.05, 1536 .. 2047 1.00, 2048 .. 3071 0.96 with full and 1.07 with half-full last tiles; up to 200
// tiles 1.16 .. 1.20, 200 .. 300 1.09 .. 1.13, 300 .. 400 0.98.
// (All of that with one tile per block.  With loads that run on across a block's tiles of 256 columns, 40 forward layers of
// 100 .. 18000 rows per expert again with each tile in each GEMM: a tile other than the rule's takes 0.85 .. 1.5 of its time, and no
// moved line is better than 0.98 in the mean.)
inline void choose_w4_tile(int64_t rows, int E, int N, int K, GemmPlan *gp)
{
    const int64_t tiles256 = (rows / 256 + E / 2) * ((N + 255) / 256);
    const int64_t tiles128 = (rows / 128 + E / 2) * ((N + 127) / 128);
    const double stages = (K + 63) / 64;
    const double t256 = static_cast<double>((tiles256 + 255) / 256) * (stages * (tiles256 > 256 ? 1.5 : 1.25) + 10.0);
    const double t128 = static_cast<double>((tiles128 + 511) / 512) *
                        (stages * (tiles128 > 256 ? 0.85 : 0.55) * (K % 64 != 0 ? 1.7 : 1.0) + 3.0);
    const bool many = tiles256 >= 768;
    if (many ? K >= 1024 || K < 256 : t256 < t128) {
        gp->bm = gp->bn = 256;
        gp->concurrent = 32;
    } else if (K >= 3072 && tiles128 > 400) {
        gp->bm = 128;
        gp->bn = 256;
        gp->concurrent = 32;
    } else {
        gp->bm = gp->bn = 128;
        gp->concurrent = 64;
    }
    gp->w4 = true;
}
// A long contraction and no more tiles of 128 x 128 than compute units, however the rows are spread: the launch takes
// as long as its weights take to arrive, and a unit's block has five stages on their way (GemmPlan::deep).
inline bool few_long_tiles(int64_t rows, int E, int N, int K)
{
    return K >= 1920 && (rows / 128 + E) * ((N + 127) / 128) <= 256;
}
// The tile is chosen for the tokens that one of n_launches FFN launches has on average, the list bounded for
// `tokens`, the most that one has.
GemmPlan choose_gemm_plan(const moe_shape &s, int which, int n_launches, int64_t tokens);
void expert_gemm_kernel_name(const moe_shape &s, int which, char *name, size_t len);

// Where each piece of the caller's workspace lives.
struct Workspace {
    int32_t *seg_cnt;      // [nseg][kMaxExperts] per-segment expert counts -> bases
    WorkItem *items[2];    // per GEMM: [n_groups][gp.max_items]
    void *hidden;          // [max_rows][d_ff] hidden activations
    GemmPlan gp[2];
    int32_t nseg;
    int32_t seg_tok;       // tokens per segment (route_segment_tokens)
    size_t bytes;
};
// For n_groups FFN launches (work lists) over n_chunks chunks.
bool layout_workspace(const moe_shape &s, int n_chunks, int n_groups, void *base, Workspace *w);

// Optional per-stage timing (moe_profile_enable): when a stage is enabled, its
// launches are bracketed by a pair of timing events on the stream they run on.
enum Stage { kStageRoute = 0, kStagePlan, kStageTiles, kStageScatter, kStageGemm1, kStageGemm2,
             kStageCombine,
             // backward pass: the five GEMMs (each one kernel), and everything else
             kStageBwdRecompute, kStageBwdDP, kStageBwdDxe, kStageBwdWgrad2, kStageBwdWgrad1,
             kStageBwdOther, kNumStages };
// Tokens per block of the gate kernel for this shape = tokens per segment of the plan.
int route_segment_tokens(const moe_shape &s);
bool prof_enabled();               // any stage is timed
enum Path { kPathSideWeightGrads = 0, kPathPulledWeights, kNumPaths };
void count_path_call(Path path);   // moe_path_calls
void prof_begin(int stage, hipStream_t st);
void prof_end(int stage, hipStream_t st);
// For a stage that is one kernel: the pair of events to attach to that kernel's own
// dispatch (hipExtLaunchKernelGGL), which then carry the kernel's begin and end
// timestamps without the launch gaps around it.  Both null when the stage is not timed.
void prof_kernel_events(int stage, hipEvent_t *start, hipEvent_t *stop);

// ---- kernel launchers (each only enqueues on `st`) ---------------------------
// when seg_cnt is not NULL the per-segment expert histogram of the dispatch plan is
// produced in the same pass
moe_status launch_gate_grad(const moe_shape &s, int t0, int t1, const uint16_t *x, const float *Wgp,
                            const float *bias, int bias_stride, const int32_t *expert_idx,
                            const float *dgate, float *dz, hipStream_t st);
moe_status launch_route(const moe_shape &s, const void *x, const void *Wg,
                        const float *bias, int bias_stride, int32_t *expert_idx,
                        float *gate, int32_t *seg_cnt, hipStream_t st);
// counted = the per-segment histogram is already in w.seg_cnt (launch_route made it);
// n_chunks == 1 also builds the GEMM work lists (otherwise launch_items does, after the ranks)
// padded: slot = e * capacity + rank (the equal-split layout) instead of offsets[e] + rank;
// offsets still receives the compact scan, and no work lists are built
// x, xe, packed: when all three are given and the plan is short enough for one launch, that
// launch also copies every token row to its kept slots (what launch_scatter does for all
// tokens) and sets *packed; otherwise *packed = false and the caller runs launch_scatter
moe_status launch_plan(const moe_shape &s, const int32_t *expert_idx, int32_t *counts,
                       int32_t *offsets, int32_t *slot_of, int32_t *src_of,
                       const Workspace &w, bool counted, int n_chunks, hipStream_t st,
                       bool padded = false, const void *x = nullptr, void *xe = nullptr,
                       bool *packed = nullptr);
// work lists of the padded layout, one per micro-op (slot positions [m*C/n, (m+1)*C/n))
moe_status launch_items_padded(const moe_shape &s, int n_micro, const int32_t *counts,
                               const Workspace &w, hipStream_t st);
// one pair of work lists per FFN group (a run of consecutive chunks, ffn_groups() of them)
moe_status launch_items(const moe_shape &s, int n_chunks, int n_groups, const int32_t *offsets,
                        const int32_t *src_of, const Workspace &w, hipStream_t st);
// How many expert-FFN launches a layer cut into n_chunks gets.  Every FFN launch streams the
// weights of all experts once, so a launch needs enough rows per expert to pay for that.
int ffn_groups(const moe_shape &s, int n_chunks);
// w.items[g] sized for E lists: list e = the output tiles of expert e alone
moe_status launch_items_per_expert(const moe_shape &s, const int32_t *offsets, const Workspace &w,
                                   hipStream_t st);
moe_status launch_scatter(const moe_shape &s, const void *x, const int32_t *slot_of,
                          void *xe, int t0, int t1, hipStream_t st);
// rows: rows of ye (slots at or beyond it are never followed); < 0 = moe_max_rows
// ye: the expert outputs in their stored type (fp16 for bf16 layers, fp32 for fp32 layers)
moe_status launch_combine(const moe_shape &s, const void *ye, const int32_t *slot_of,
                          const float *gate, float *y, void *y_act, int t0, int t1,
                          hipStream_t st, int64_t rows = -1);
// pre: NULL, or fp16 [rows, d_ff] receiving the pre-activations of the first GEMM (bf16 layers)
// row_src: NULL, or the dispatch plan's src_of: `xe` is then the token matrix x itself and the
// first GEMM gathers slot i's row from token src_of[i] / k (bf16 layers)
moe_status launch_ffn(const moe_shape &s, const void *xe, const void *W1p,
                      const float *b1, const void *W2p, const float *b2, void *ye,
                      const Workspace &w, int chunk, hipStream_t st, void *pre = nullptr,
                      const int32_t *row_src = nullptr);
// bytes per element of the expert outputs ye
inline int ye_elem_bytes(const moe_shape &s) { return s.dtype == MOE_BF16 ? 2 : 4; }
moe_status launch_pack(const moe_shape &s, const void *W1, const void *W2, void *W1p,
                       void *W2p, hipStream_t st);

// ---- device helpers --------------------------------------------------------
#if defined(__HIPCC__)
__device__ __forceinline__ float bf16_to_f32(uint16_t b)
{
    return __uint_as_float(static_cast<uint32_t>(b) << 16);
}
// round to nearest, ties to even; finite inputs
__device__ __forceinline__ uint16_t f32_to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return static_cast<uint16_t>(u >> 16);
}
// Order of the packed gate matrix inside a run of 16 columns: position 4 g + i holds column
// 4 i + g (its own inverse), so that 16 bytes are what a 16-lane group g of the gate kernel's
// matrix instruction needs for four steps.
__host__ __device__ __forceinline__ int packed_gate_column(int i)
{
    return (i & ~15) | ((i & 3) << 2) | ((i >> 2) & 3);
}
__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }
#endif

}  // namespace moe
