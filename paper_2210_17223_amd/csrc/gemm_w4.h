// The tile GEMMs on four wavefronts: what its kernels share.  Included inside the
// translation unit's own namespace; the loop itself is gemm_w4_body.inc, included in the body
// of every kernel that runs it for one tile (the forward's 128 x 128 tiles, the backward's row GEMMs), each
// with an epilogue of its own, and gemm_w4_run.h's for the forward's other tiles.
#pragma once

#include <type_traits>
#include <utility>

// ---------------------------------------------------------------- GEMM tiles, four wavefronts
// 256 x 256 output tiles, 64-deep stages, one wavefront per SIMD:
//  * four wavefronts of 128 x 128 (2 x 2) of 16 x 16 x 32 matrix instructions, the 64
//    accumulators of a wavefront (256 registers) pinned to AGPRs; an operand fragment read from
//    LDS feeds eight of them.
//  * Operands go from global memory straight into LDS (16-byte buffer loads to LDS: no staging
//    registers, no LDS write instructions) through a ring of five 32 KiB units (256 rows x 64 deep
//    of one operand), all 160 KiB of it: while stage k is multiplied, the token rows of stage
//    k + 2 and the weights of stage k + 1 .. k + 2 are on their way.  A unit is written linearly,
//    1 KiB per instruction, so the 16-byte pieces of a row are XOR-swizzled with the row on the
//    global side: fragment reads are free of bank conflicts.
//  * One barrier per stage, in its middle: behind it the next stage's fragments are read while
//    the second half is multiplied, and the finished stage's units are refilled.  The last two stages have
//    nothing to refill them with: dP's GEMM brings its tile of pre-activations into the four units that
//    come free, 128 KiB of fp16 for 256 x 256 values, and its epilogue turns them into dP in their places.  Behind
//    the loop, a line at a time through registers, that tile was 480 us of 2497 (63622 rows, N = 8192, K = 2048: 2012
//    now; 8192 rows, 768 x 3072 on 128 x 128 tiles: 92 -> 75).  The other GEMMs load nothing there, where they used to
//    load the last stage again: 82.3 -> 81.4, 56.2 -> 54.6, 117 -> 106 us of the GEMMs of that size.
//  * Every memory instruction is issued singly between two matrix instructions in a fixed order;
//    those are inline assembly so that the accumulators stay in AGPRs and the order holds.
//    Neighbouring ones share an operand (serpentine order).
// What bounds it: the matrix cores are busy for 65 % / 77 % of the cycles (N = 8192, K = 2048, GeLU / N =
// 2048, K = 8192; with one tile per block 62 / 79), at a clock of 1.75 / 1.71 GHz that the chip sets by the energy per
// operation (on all-ones operands the same launches are 21 % faster).  With 32 x 32 x 16 instructions and operands staged
// through registers it was 56 % / 78 % at 1.68 / 1.55 GHz: the first GEMM lost cycles, the second takes as many
// as before and they have become cheaper.  On 64 x 1024 rows alone, after thirty launches, with a block's loads
// running on from tile to tile (gemm_w4_run.h): 1790 / 1600 us, of which the matrix instructions and barriers by themselves
// take 1333 / 1101, and the loads into LDS beside them 30 % / 41 % on top; a vendor library's dense products
// of these sizes 1540 / 1515.  (After two launches, while the clock still follows the load, 15 % more.)
// Loads into LDS run at 9 to 10 TB/s over the chip beside the matrix instructions, whatever the tile.
// 128 x 256 (64 x 128 per wavefront) and 128 x 128 tiles (64 x 64) run the same loop.  128 x 256 has
// LDS for three whole stages instead of the ring; of 128 x 128 a compute unit holds two blocks, one
// of which multiplies through the other's prologue and epilogue.  Against 32 x 32 x 16 tiles staged
// through registers, 8192 rows, 16 experts, us: N = 3072, K = 768 72.6 -> 57.7 (128 x 128); N = 768,
// K = 3072 55.8 -> 40.8 (128 x 256).
// Where a launch has few rows per expert and no more 128 x 128 tiles than there are compute units, a unit holds one
// block with five whole stages (160 KiB) instead: such a launch is bound by the bytes that are on their way.  8 experts of
// 64 rows, N = 2048, K = 7168 (235 MB of weights): 92.2 -> 72.3 us, 2.5 -> 3.2 TB/s.
// Operand addresses are 32-bit byte offsets into two buffer resources (the tile's rows, or
// the whole token matrix when the rows are gathered through row_src; the expert's weight
// matrix), which the host checks fit.
constexpr size_t w4_lds(int bm, int bn) { return (bm == bn ? 5 * bm : 3 * (bm + bn)) * 128; }
constexpr size_t kW4Lds = w4_lds(256, 256);
// Blocks whose loads run on from tile to tile (gemm_w4_run.h, the weight gradients) have a compute unit to themselves, so
// kRunUnits of them run at once.  A share of the tiles ends after kRunStages stages of 64, 0.2 ms, which is one tile of the large
// layer's second GEMM: the unit then goes to whoever waits.  Median / longest time of a decode step (five launches) on another
// stream beside large layers (32768 tokens, 2048 x 8192, 64 experts) with a launch's tiles in 256 shares, us: 1640 / 3500, of a layer
// of 4096 tokens, 768 x 3072: 3660 / 3780; in shares of 64 stages 365 / 900 and 680 / 1150, of 128 430 / 1050 and 780 / 1350, of 256 500 /
// 1930 and 1700 / 2200; one tile per block 280 / 1100 and 535 / 1250.  What the shares' ends cost: the large layer 1.01 with 64
// stages, 1.003 with 128, its training step 1.04, 1.012 and 1.004 with 256; four other forward layers 1.000 .. 1.006, eight training
// steps whose weight gradients run beside the other GEMMs 0.97 .. 1.00, since these get in between the shares, too.
constexpr int kRunUnits = 256, kRunStages = 128;

#define MOE_LGKM0() asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory")
#define MOE_VMCNT(n) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(n) : "memory")
#define MOE_SB() __builtin_amdgcn_sched_barrier(0)
#define MOE_BAR()                                                                                 \
    do {                                                                                         \
        MOE_SB();                                                                                \
        __builtin_amdgcn_s_barrier();                                                            \
        MOE_SB();                                                                                \
    } while (0)

// The compiler puts no wait states around inline assembly.  WAIT: two of them, what a vector
// instruction's result needs before a matrix instruction reads it, in the same statement, so that
// nothing gets in between (for the first one behind a conversion).  That nothing else comes too
// close, registers moved on the way round a loop among it, tests/test_matrix_hazards.py reads
// back from the built library.  (Two wait states at the top of every stage: gpt2s-sized layers, 8192
// rows of 768 x 3072, 61.5 -> 61.9 us in the first GEMM.)
// ZERO: the accumulator starts at zero.
template <bool F16, bool WAIT, bool ZERO = false>
__device__ __forceinline__ void mfma_16x16x32_agpr(f32x4 &acc, const u32x4 &a, const u32x4 &b)
{
    static_assert(!(F16 && WAIT), "no caller converts to fp16");
    if constexpr (F16 && ZERO)
        asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, 0" : "=a"(acc) : "v"(a), "v"(b));
    else if constexpr (F16)
        asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
    else if constexpr (ZERO && WAIT)
        asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc) : "v"(a), "v"(b));
    else if constexpr (ZERO)
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc) : "v"(a), "v"(b));
    else if constexpr (WAIT)
        asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
    else
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

// Behind the last matrix instruction: the results have left the pipeline after the no-ops, and the
// fence keeps reads of the accumulators behind them.
#define MOE_MATRIX_RESULTS()                                                                     \
    do {                                                                                         \
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");                                       \
        MOE_SB();                                                                                \
    } while (0)

// 16 bytes per lane from base + voff + soff to LDS at `at` + 16 * lane.  Written out because
// behind the compiler's builtin every later LDS read waits for all loads; completion is counted
// by hand (MOE_VMCNT).  The range check that turns a load into zeros sees voff only.
__device__ __forceinline__ void load_to_lds(__amdgpu_buffer_rsrc_t rs, int voff, uint32_t at, int soff)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %3 offen lds"
                 ::"v"(voff), "s"(rs), "s"(at), "s"(soff) : "memory", "m0");
#endif
}
// The dword at p, and behind its load N of load_to_lds's, at `at`, `at` + 1024, ..., that are still on
// their way afterwards.  One asm block: `v` is not a register with a load in flight where the compiler may
// move or copy it.
template <int N>
__device__ __forceinline__ void load_dword_before(int &v, const int32_t *p, __amdgpu_buffer_rsrc_t rs,
                                                  const int (&voff)[N], uint32_t at)
{
    static_assert(N == 4 || N == 8, "written out for these");
#if defined(__HIP_DEVICE_COMPILE__)
#define MOE_NEXT(o) "s_add_u32 m0, m0, 0x400\n\ts_nop 0\n\tbuffer_load_dwordx4 %" #o ", %2, 0 offen lds\n\t"
#define MOE_FIRST "global_load_dword %0, %1, off\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %4, %2, 0 offen lds\n\t"
    if constexpr (N == 4)
        asm volatile(MOE_FIRST MOE_NEXT(5) MOE_NEXT(6) MOE_NEXT(7) "s_waitcnt vmcnt(4)"
                     : "=&v"(v)
                     : "v"(p), "s"(rs), "s"(at), "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3])
                     : "memory", "m0", "scc");
    else
        asm volatile(MOE_FIRST MOE_NEXT(5) MOE_NEXT(6) MOE_NEXT(7) MOE_NEXT(8) MOE_NEXT(9) MOE_NEXT(10)
                         MOE_NEXT(11) "s_waitcnt vmcnt(8)"
                     : "=&v"(v)
                     : "v"(p), "s"(rs), "s"(at), "v"(voff[0]), "v"(voff[1]), "v"(voff[2]), "v"(voff[3]),
                       "v"(voff[4]), "v"(voff[5]), "v"(voff[6]), "v"(voff[7])
                     : "memory", "m0", "scc");
#undef MOE_FIRST
#undef MOE_NEXT
#endif
}
__device__ __forceinline__ uint32_t lds_address(const void *p)
{
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const void *)p));
}

template <int... I, typename F>
__device__ __forceinline__ void static_for_each(std::integer_sequence<int, I...>, F f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F f)
{
    static_for_each(std::make_integer_sequence<int, N>{}, f);
}
