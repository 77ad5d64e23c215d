// Expert FFN with host-resident expert weights (paper Sec. 4.2 "Expert packing":
// DRAM-offloading; Sec. 6.2: packed experts are loaded and computed one at a time).
// Expert e's packed weights travel host -> staging slot e % resident on a copy stream
// while earlier experts are computed; the two GEMMs of expert e then run on the caller's
// stream from a work list that holds expert e's tiles only.  Bound by the host link:
// 2 d h element bytes per expert against a few microseconds of matrix-core work per row.
// Page-locked weights are read over the link by a kernel, both matrices of an expert in one
// launch, the experts on two streams in turn; others go through the runtime's copy.
#include "common.h"
#include "moe_offload.h"

#include <mutex>

namespace moe {
namespace {

struct OffloadResources {
    hipStream_t copy[2] = {};               // experts take turns if their weights are page-locked
    hipEvent_t ready[kMaxExperts] = {};     // slot filled
    hipEvent_t freed[kMaxExperts] = {};     // slot's expert computed
    hipEvent_t begin = nullptr;
    bool ok = false;
    std::mutex enqueue;                     // held while a call enqueues on the copy streams
};
OffloadResources g_res[16];
std::mutex g_res_mutex;

moe_status resources(OffloadResources **out)
{
    int dev = 0;
    MOE_TRY_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= 16) {
        set_error("device ordinal %d is outside the supported range", dev);
        return MOE_EUNSUPPORTED;
    }
    std::lock_guard<std::mutex> lock(g_res_mutex);
    OffloadResources &r = g_res[dev];
    if (!r.ok) {
        for (hipStream_t &c : r.copy) MOE_TRY_HIP(hipStreamCreateWithFlags(&c, hipStreamNonBlocking));
        MOE_TRY_HIP(hipEventCreateWithFlags(&r.begin, hipEventDisableTiming));
        for (int i = 0; i < kMaxExperts; ++i) {
            MOE_TRY_HIP(hipEventCreateWithFlags(&r.ready[i], hipEventDisableTiming));
            MOE_TRY_HIP(hipEventCreateWithFlags(&r.freed[i], hipEventDisableTiming));
        }
        r.ok = true;
    }
    *out = &r;
    return MOE_OK;
}

bool supported(const moe_shape *s)
{
    return s != nullptr && s->dtype == MOE_BF16 && s->T >= 1 && s->E >= 1 && s->E <= kMaxExperts &&
           s->k >= 1 && s->k <= kMaxTopK && s->k <= s->E && s->capacity >= 1 && s->d_model >= 8 &&
           s->d_ff >= 8 && s->d_model % 8 == 0 && s->d_ff % 8 == 0;
}

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

// One expert's two weight matrices, n 16-byte vectors each, from page-locked host memory to its
// slot; an expert without rows (offsets) is not read.  The link is full with some 64 KiB of reads in
// flight, so few blocks do: GB/s of back-to-back launches of 16 MiB with 8 / 16 / 64 / 256 blocks 56.1 /
// 56.6 / 56.2 / 52.0, the runtime's copy 55.4; behind an event that another stream records after
// every copy, as here, the runtime's copies of 8 MiB reach 37 to 41: what a copy engine's start and
// end signals cost beside 0.15 ms of transfer, a kernel's launch does not.  256 tokens, 16 experts
// of 1024 x 4096, two slots: 6120 -> 5040 us.  On two streams in turn the link is not idle between one
// expert's event and the next one's launch either: 5030 -> 4870 us, 55 GB/s.
constexpr int kPullBlocks = 16;
__global__ __launch_bounds__(256) void pull_weights_kernel(
    const u32x4 *__restrict__ h1, const u32x4 *__restrict__ h2, u32x4 *__restrict__ d1,
    u32x4 *__restrict__ d2, size_t n, const int32_t *__restrict__ offsets, int expert)
{
    if (offsets[expert] == offsets[expert + 1]) return;
    constexpr int U = 4;                         // loads in flight per lane
    const size_t step = static_cast<size_t>(gridDim.x) * (256 * U);
    for (int m = 0; m < 2; ++m) {
        const u32x4 *src = m == 0 ? h1 : h2;
        u32x4 *dst = m == 0 ? d1 : d2;
        for (size_t i = static_cast<size_t>(blockIdx.x) * (256 * U) + threadIdx.x; i < n; i += step) {
            u32x4 v[U];
#pragma unroll
            for (int q = 0; q < U; ++q)          // (past the end: the last vector again, not stored)
                v[q] = src[i + q * 256 < n ? i + q * 256 : n - 1];
#pragma unroll
            for (int q = 0; q < U; ++q)
                if (i + q * 256 < n) dst[i + q * 256] = v[q];
        }
    }
}

// The device's address of `bytes` of page-locked host memory at p, or NULL if the device cannot read
// all of them in place (pageable memory, or not inside one allocation: the host's and the device's
// addresses are often the same, so two ends that both map say nothing about the bytes between them).
const char *device_view(const void *p, size_t bytes)
{
    hipPointerAttribute_t a{};
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();                 // an unknown address is no error here
        return nullptr;
    }
    if (a.type != hipMemoryTypeHost || a.devicePointer == nullptr) return nullptr;
    if (hipMemGetAddressRange(&base, &size, a.devicePointer) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    const char *view = static_cast<const char *>(a.devicePointer);
    const size_t at = reinterpret_cast<uintptr_t>(view) - reinterpret_cast<uintptr_t>(base);
    return at <= size && bytes <= size - at && (reinterpret_cast<uintptr_t>(view) & 15u) == 0 ? view : nullptr;
}

size_t expert_bytes(const moe_shape &s) { return static_cast<size_t>(s.d_model) * s.d_ff * 2; }

void layout(const moe_shape &s, void *base, Workspace *w)
{
    char *p = static_cast<char *>(base);
    size_t off = 0;
    *w = Workspace{};
    for (int g = 0; g < 2; ++g) {
        w->gp[g] = choose_gemm_plan(s, g, 1, s.T);          // the resident path's tile shapes
        w->items[g] = reinterpret_cast<WorkItem *>(p + off);
        off += align_up(static_cast<size_t>(s.E) * w->gp[g].max_items * sizeof(WorkItem), 256);
    }
    w->hidden = p + off;
    off += align_up(static_cast<size_t>(moe_max_rows(&s)) * s.d_ff * 2, 256);
    w->bytes = off;
}

}  // namespace
}  // namespace moe

using namespace moe;

extern "C" {

size_t moe_offload_staging_bytes(const moe_shape *s, int32_t resident)
{
    if (!supported(s) || resident < 1) return 0;
    return static_cast<size_t>(resident > s->E ? s->E : resident) * 2 * align_up(expert_bytes(*s), 256);
}

size_t moe_offload_workspace_bytes(const moe_shape *s)
{
    if (!supported(s)) return 0;
    Workspace w;
    layout(*s, reinterpret_cast<void *>(static_cast<uintptr_t>(256)), &w);
    return w.bytes;
}

moe_status moe_expert_ffn_offloaded(const moe_shape *s, const void *xe, const int32_t *offsets,
                                    const void *W1p_host, const void *W2p_host, const float *b1,
                                    const float *b2, void *ye, void *staging, int32_t resident,
                                    void *workspace, void *stream)
{
    if (!supported(s)) {
        set_error("moe_expert_ffn_offloaded: bf16 layers, E <= %d, k <= %d, d_model and d_ff "
                  "multiples of 8", kMaxExperts, kMaxTopK);
        return s == nullptr ? MOE_EINVAL : MOE_EUNSUPPORTED;
    }
    if (resident < 1) {
        set_error("resident = %d: at least one expert slot is needed", resident);
        return MOE_EINVAL;
    }
    const void *need[] = {xe, offsets, W1p_host, W2p_host, ye, staging, workspace};
    for (const void *p : need) {
        if (p == nullptr || (reinterpret_cast<uintptr_t>(p) & 15u) != 0) {
            set_error("moe_expert_ffn_offloaded: a required pointer is NULL or not 16-byte aligned");
            return MOE_EINVAL;
        }
    }
    if (resident > s->E) resident = s->E;
    OffloadResources *r = nullptr;
    const moe_status rs = resources(&r);
    if (rs != MOE_OK) return rs;
    // one call at a time enqueues on this device's copy streams and shared events
    std::lock_guard<std::mutex> enqueue(r->enqueue);
    Workspace w;
    layout(*s, workspace, &w);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const size_t eb = expert_bytes(*s), slot_bytes = align_up(eb, 256);
    char *stage = static_cast<char *>(staging);
    const char *h1 = static_cast<const char *>(W1p_host), *h2 = static_cast<const char *>(W2p_host);
    const char *v1 = device_view(h1, eb * s->E), *v2 = device_view(h2, eb * s->E);
    const bool pull = v1 != nullptr && v2 != nullptr;
    if (pull) count_path_call(kPathPulledWeights);

    moe_status rc = launch_items_per_expert(*s, offsets, w, st);
    if (rc != MOE_OK) return rc;
    // a copy stream may not touch the staging area before what the caller enqueued earlier
    // (possibly a previous call's GEMMs reading it) has finished
    MOE_TRY_HIP(hipEventRecord(r->begin, st));
    for (int e = 0; e < s->E; ++e) {
        const int slot = e % resident;
        char *d1 = stage + static_cast<size_t>(slot) * 2 * slot_bytes, *d2 = d1 + slot_bytes;
        hipStream_t copy = r->copy[pull ? e % 2 : 0];
        if (e < (pull ? 2 : 1)) MOE_TRY_HIP(hipStreamWaitEvent(copy, r->begin, 0));
        if (e >= resident) MOE_TRY_HIP(hipStreamWaitEvent(copy, r->freed[slot], 0));
        const size_t at = static_cast<size_t>(e) * eb;
        if (pull) {
            hipLaunchKernelGGL(pull_weights_kernel, dim3(kPullBlocks), dim3(256), 0, copy,
                               reinterpret_cast<const u32x4 *>(v1 + at), reinterpret_cast<const u32x4 *>(v2 + at),
                               reinterpret_cast<u32x4 *>(d1), reinterpret_cast<u32x4 *>(d2), eb / 16, offsets, e);
            MOE_TRY_HIP(hipGetLastError());
        } else {
            MOE_TRY_HIP(hipMemcpyAsync(d1, h1 + at, eb, hipMemcpyHostToDevice, copy));
            MOE_TRY_HIP(hipMemcpyAsync(d2, h2 + at, eb, hipMemcpyHostToDevice, copy));
        }
        MOE_TRY_HIP(hipEventRecord(r->ready[slot], copy));
        MOE_TRY_HIP(hipStreamWaitEvent(st, r->ready[slot], 0));
        // The GEMM kernel addresses expert e's weights as base + e * d * h elements: hand it
        // a base that lands on the slot.  Only [slot, slot + eb) is ever dereferenced, since
        // list e holds expert e's tiles only.
        const char *f1 = d1 - static_cast<size_t>(e) * eb, *f2 = d2 - static_cast<size_t>(e) * eb;
        rc = launch_ffn(*s, xe, f1, b1, f2, b2, ye, w, e, st);
        if (rc != MOE_OK) return rc;
        MOE_TRY_HIP(hipEventRecord(r->freed[slot], st));
    }
    return MOE_OK;
}

}  // extern "C"
