// Tiles of 256 columns: a block, which has a compute unit to itself, works through a share of the tiles and its loads
// run on from tile to tile.  Included behind gemm_w4.h, inside the translation unit's own namespace.
//
// The stages are those of gemm_w4_body.inc.  Its last ones have no operands of their tile left to ask for: here
// they ask for the next tile's first ones, whose fragments the last stage reads, so that the next tile's
// first matrix instruction stands right behind the epilogue.  Before that every tile began with an
// empty ring, the wait for its work item, its rows' indices and two stages of loads, and its block
// ended with every store accepted.
//  * 256 x 256 (BM = 256): the ring of five units of 32 KiB; when the last stage is through, four hold the next
//    tile's first two stages and the fifth is free for the epilogue.
//  * 128 x 256 (BM = 128): three whole stages of 48 KiB, all on their way for the next tile, and 16 KiB beside them
//    for the epilogue.
// A tile leaves through a quarter of those per wavefront, UR rows of 128 values at a time, the 16-byte pieces of a
// row XOR-swizzled with the row.  LDS takes a wavefront's accesses in order and no other wavefront touches its
// quarter (loads into it are its own, too), so nothing is waited for.
// Measured, us, one tile per block before / a share of the tiles per block: 64 x 1024 rows alone, N = 8192, K = 2048,
// GeLU 1856 -> 1773, N = 2048, K = 8192 1589 -> 1586 (its tiles are of 128 stages; on all-ones operands, at the higher clock,
// 1575 -> 1455 and 1317 -> 1316); with the pre-activations kept, 63622 rows 2087 -> 1877; of Zipf(1.2)-distributed rows the layer of
// 16384 tokens, 1024 x 4096, 32 experts 375 -> 362; of 3001 tokens, 1000 x 2600, 13 experts, all options 191 -> 179.  Prologue,
// barriers and epilogue of the first product take 176 of its 1773 by themselves (313 of 1856).  These with all of a launch's
// tiles in 256 shares; in shares of kRunStages 1790 and 1600, 230 of 1790.
// What runs beside such a launch: a block holds its unit until its share is done, all of its LDS and 440 or 448 of the 512 registers
// of every SIMD (256 x 256; at most 472 with the pre-activations kept; 272 to 312 on 128 x 256).  Wavefronts of another stream
// that ask for no LDS and for the rest of the registers get in, as the pack (32) and the stand-in link's copy (40) do; what
// needs LDS (gate, plan) or more registers waits for the end of a share (kRunStages).
// Three items are known ahead: the tile's, the next one's, whose rows' offsets are in registers, and the
// one's behind it, whose rows' indices are on their way during a whole tile.

constexpr size_t kW4RunLds = 160 * 1024;
// tiles of a block's share (a stage of 128 x 256 takes half as long as one of 256 x 256)
inline int w4_run_share(int bm, int K) { return std::max(1, kRunStages * 256 / bm / std::max((K + 63) / 64, 4)); }
// blocks of a launch: blocks 256 g .. 256 g + 255 take the entries from 256 g * share on, each every 256th
inline int w4_run_blocks(int entries, int share)
{
    const int whole = (entries - 1) / (kRunUnits * share);
    return whole * kRunUnits + std::min(entries - whole * kRunUnits * share, kRunUnits);
}

template <int BM>
struct W4Place {                       // where a wavefront stands in its tile
    char *patch;                       // its quarter of the free LDS: UR rows of 256 bytes
    int lane, wm, wn, fr, oct;
    static constexpr int UR = BM / 8, TM = BM / 32, TN = 8;
    // a lane's four values of column block i (16 columns) of a row block, as 16-bit values, the patch's 16 rows `part`
    __device__ __forceinline__ char *at(int i, int part) const
    {
        const int row = part * 16 + fr;
        return patch + row * 256 + (((2 * i + (oct >> 1)) ^ fr) << 4) + (oct & 1) * 8;
    }
    // the patch's rows from 16 part on, whole lines of 16-bit values, to a [rows, N] matrix: rows r .. r + R - 1 of the
    // wavefront's part of the tile
    template <int R>
    __device__ __forceinline__ void leave(uint16_t *out, const WorkItem &item, int r, int part, int N) const
    {
        const int row0 = item.row0 + wm * (BM / 2) + r, col0 = item.n0 + wn * 128;
        // (a row past the tile's or a column past N lies past the resource)
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            out + static_cast<size_t>(row0) * N, 0, static_cast<unsigned>(max(item.row1 - row0, 0)) * N * 2u, 0x00020000);
        const int col = col0 + lane % 16 * 8;
        const int first = col < N ? (lane / 16 * N + col) * 2 : 0x7ff00000, step = col < N ? N * 8 : 0;
        MOE_SB();
#pragma unroll
        for (int it = 0; it < R / 4; ++it) {
            const int row = it * 4 + lane / 16;
            const u32x4 q = *reinterpret_cast<const u32x4 *>(patch + (part * 16 + row) * 256 + ((lane % 16 ^ (row & 15)) << 4));
            __builtin_amdgcn_raw_buffer_store_b128(q, rs, first + it * step, 0, 0);
            if (it % 4 == 3) MOE_SB();
        }
    }
};

// C tile += A[rows of the work item, K] . W[expert][n0 .. n0 + 255, K]^T for `share` items, every 256th from the block's
// first one on (a multiple of eight: the XCD of an entry stays what the list was made for).  F16: fp16
// rather than bf16 operands.  KTAIL: K is not a multiple of 64, or below four stages; what lies past it reads as zeros.
// ABL: see grouped_gemm_w4_kernel.  epilogue(acc, prepare(item, wn, oct), item, place, landed) takes the finished tile out of
// the accumulators, without a branch, acc[i][j][c] = column wn * 128 + i * 16 + oct * 4 + c, row wm * BM / 2 + j * 16 + fr, and calls landed() once, in
// front of its first store: what the next tile waits for early has to be there before stores stand in front of it.
template <bool F16, bool KTAIL, int BM, int ABL, typename Prepare, typename Epilogue>
__device__ __forceinline__ void w4_run(const uint16_t *__restrict__ A, const uint16_t *__restrict__ W,
                                       const WorkItem *__restrict__ items, const int32_t *__restrict__ nitems, int entries, int share,
                                       int N, int K, const int32_t *__restrict__ row_src, int row_div, int a_rows,
                                       Prepare prepare, Epilogue epilogue)
{
    constexpr int TM = BM / 32, TN = 8, BK = 64;
    constexpr bool RING5 = BM == 256;
    constexpr int A_UNIT = BM * 128, W_UNIT = 256 * 128;
    constexpr int AR = BM / 4;                    // rows of A that a wavefront loads
    constexpr int stride = kRunUnits;
    int b = blockIdx.x / stride * stride * share + blockIdx.x % stride;
    const int stop = min(entries, b + share * stride);
    auto item_at = [&](int b) {
        WorkItem t{-1, 0, 0, 0};
        int at = b < stop ? b : -1;
        if (nitems != nullptr && at >= 0) {
            const int total = *nitems, per_xcd = (total + 7) / 8, slot = b / 8;
            at = b % 8 * per_xcd + slot;
            if (slot >= per_xcd || at >= total) at = -1;
        }
        if (at >= 0) t = items[at];
        t.expert = __builtin_amdgcn_readfirstlane(t.expert);    // (the same for all lanes: scalars)
        t.row0 = __builtin_amdgcn_readfirstlane(t.row0);
        t.row1 = __builtin_amdgcn_readfirstlane(t.row1);
        t.n0 = __builtin_amdgcn_readfirstlane(t.n0);
        return t;
    };
    WorkItem item = item_at(b), next = item_at(b + stride);
    if (item.expert < 0) return;

    extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
    char *const lds = reinterpret_cast<char *>(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1, fr = lane & 15, oct = lane >> 4;
    const int KT = max((K + BK - 1) / BK, 4);

    // operands of a tile; of none: no byte is in range, and loads leave zeros without going to memory
    auto rows_of = [&](const WorkItem &t) {
        const uint16_t *at = row_src != nullptr || t.expert < 0 ? A : A + static_cast<size_t>(t.row0) * K;
        const unsigned n = t.expert < 0 ? 0u : static_cast<unsigned>(row_src != nullptr ? a_rows : t.row1 - t.row0);
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(at), 0, n * static_cast<unsigned>(K) * 2u, 0x00020000);
    };
    auto weights_of = [&](const WorkItem &t) {
        const uint16_t *at = t.expert < 0 ? W : W + (static_cast<size_t>(t.expert) * N + t.n0) * K;
        const unsigned n = t.expert < 0 ? 0u : static_cast<unsigned>(N - t.n0);
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(at), 0, n * static_cast<unsigned>(K) * 2u, 0x00020000);
    };
    // load q of this wavefront's TM (TN) of a unit: rows wave * AR (64) + 8 q .. + 7, eight 16-byte pieces
    // each; lane l lands at row l / 8, place l % 8, where piece place ^ (row / 2 % 8) belongs
    int w_src[TN], a_src[TM], a_next[TM];
    int first_col[2];                             // KTAIL: the piece's first column in its stage (q even / odd)
#pragma unroll
    for (int q = 0; q < TN; ++q) {
        const int r = wave * 64 + q * 8 + (lane >> 3), piece = (lane & 7) ^ ((r >> 1) & 7);
        w_src[q] = (r * K + piece * 8) * 2;
        if (q < 2) first_col[q] = piece * 8;
    }
    // lane l's: row l of the wavefront's AR of a tile, in A or (packed rows) in the tile, -1 past its last one; from
    // there the offsets
    const int own_row = wave * AR + (lane & (AR - 1));
    auto source_at = [&](const WorkItem &t) { return row_src + t.row0 + min(own_row, t.row1 - t.row0 - 1); };
    auto row_or_none = [&](const WorkItem &t, int source) {
        return own_row < t.row1 - t.row0 ? (row_src != nullptr ? source / row_div : own_row) : -1;
    };
    auto a_offsets = [&](int row, int (&out)[TM]) {
        int here = lane;
        asm volatile("" : "+v"(here));
#pragma unroll
        for (int q = 0; q < TM; ++q) {
            const int r = q * 8 + (here >> 3);    // (wave * AR is a multiple of 16)
            const int from = __shfl(row, r);
            out[q] = ((from * K + ((here & 7) ^ ((r >> 1) & 7)) * 8) * 2) | ((from >> 31) & 0x7ffffff0);
        }
    };
    const uint32_t a_dest = lds_address(lds) + wave * (A_UNIT / 4), w_dest = lds_address(lds) + wave * (W_UNIT / 4);
    __amdgpu_buffer_rsrc_t rsa = rows_of(item), rsw = weights_of(item);
    // (a piece past K and a row past the tile's get an offset past every resource: zeros, without going to memory.
    // What is loaded, 9 to 10 TB/s into LDS over the chip, is what these loops wait for: with the tile's last row in their
    // place the layer of 16384 tokens, 1024 x 4096, 32 experts, Zipf(1.2), took 362 us, and 348 now.)
    auto piece_of = [&](int src, int q, int k) {
        if constexpr (KTAIL) return k * BK + first_col[q & 1] < K ? src : 0x7ffffff0;
        else return src;
    };
    auto load_a = [&](int q, int unit, int k) { load_to_lds(rsa, piece_of(a_src[q], q, k), a_dest + unit + q * 1024, k * (BK * 2)); };
    auto load_w = [&](int q, int unit, int k) { load_to_lds(rsw, piece_of(w_src[q], q, k), w_dest + unit + q * 1024, k * (BK * 2)); };

    // RING5: A and W of this stage, A and W of the next, and the free unit; else the A and W units of
    // this stage, the next and the one after it (uf: its A unit)
    int ua = 0, uw = A_UNIT, ua1 = A_UNIT + W_UNIT, uw1 = 2 * A_UNIT + W_UNIT, uf = 2 * (A_UNIT + W_UNIT);
    if (row_src != nullptr) {
        // the first tile's indices are fetched while its first weights are on their way
        int source = 0, w_first[TN];
#pragma unroll
        for (int q = 0; q < TN; ++q) w_first[q] = piece_of(w_src[q], q, 0);
        load_dword_before(source, source_at(item), rsw, w_first, w_dest + uw);
        a_offsets(row_or_none(item, source), a_src);
    } else {
#pragma unroll
        for (int q = 0; q < TN; ++q) load_w(q, uw, 0);
        a_offsets(row_or_none(item, 0), a_src);
    }
#pragma unroll
    for (int q = 0; q < TM; ++q) load_a(q, ua, 0);
#pragma unroll
    for (int q = 0; q < TM; ++q) load_a(q, ua1, 1);
#pragma unroll
    for (int q = 0; q < TN; ++q) load_w(q, uw1, 1);
    if constexpr (!RING5) {
#pragma unroll
        for (int q = 0; q < TN; ++q) load_w(q, uf + A_UNIT, 2);
    }

    f32x4 acc[TN][TM];
    u32x4 wf[2][TN], af[2][TM];
    if constexpr (ABL & 1) {
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.0f;
    }
    int fbase[2];                      // a lane's fragment of the two 32-deep steps inside a unit
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) fbase[ks] = fr * 128 + (((ks * 4 + oct) ^ ((fr >> 1) & 7)) << 4);
    const int aoff = wm * (A_UNIT / 2), woff = wn * (W_UNIT / 2);

    MOE_VMCNT(RING5 ? TM + TN : TM + 2 * TN);
    MOE_BAR();
    if (next.expert >= 0) {
        int source = 0;
        if (row_src != nullptr) source = *source_at(next);
        a_offsets(row_or_none(next, source), a_next);
    } else {
#pragma unroll
        for (int q = 0; q < TM; ++q) a_next[q] = a_src[q];
    }
#pragma unroll
    for (int i = 0; i < TN; ++i) wf[0][i] = *reinterpret_cast<const u32x4 *>(lds + uw + woff + fbase[0] + i * 2048);
#pragma unroll
    for (int j = 0; j < TM; ++j) af[0][j] = *reinterpret_cast<const u32x4 *>(lds + ua + aoff + fbase[0] + j * 2048);
    if constexpr (ABL & 2) {           // (the measurement variant multiplies these again and again)
#pragma unroll
        for (int i = 0; i < TN; ++i) wf[1][i] = wf[0][i];
#pragma unroll
        for (int j = 0; j < TM; ++j) af[1][j] = af[0][j];
    }

    // TM * TN matrix instructions of a 32-deep step, memory instruction m (mem) after number m; ZERO: they start the tile
    auto step = [&](auto slotc, auto zero, auto mem) {
        constexpr int s = decltype(slotc)::value;
        static_for<TM * TN>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            constexpr int j = m / TN, i = (j & 1) != 0 ? TN - 1 - m % TN : m % TN;
            if constexpr (!(ABL & 1)) mfma_16x16x32_agpr<F16, false, decltype(zero)::value>(acc[i][j], wf[s][i], af[s][j]);
            mem(mc);
            MOE_SB();
        });
    };
    // fragment read v (W first) of a step into slot s
    auto read = [&](auto slotc, auto vc, int wat, int aat) {
        constexpr int s = decltype(slotc)::value, v = decltype(vc)::value;
        if constexpr (!(ABL & 2)) {
            if constexpr (v < TN)
                wf[s][v] = *reinterpret_cast<const u32x4 *>(lds + wat + v * 2048);
            else
                af[s][v - TN] = *reinterpret_cast<const u32x4 *>(lds + aat + (v - TN) * 2048);
        }
    };
    using std::integral_constant;
    constexpr int NR = 2 * (TM + TN);            // fragment reads after matrix instructions 0, 2 .. NR - 2
    constexpr int A_GAP = BM == 256 ? 4 : 2;     // loads of A behind them
    // A stage, with the token rows of stage ka (the tile's own, or the next tile's) and the weights of stage kw on
    // their way out; wait: for the stage behind it, which what is younger need not have followed
    auto stage = [&](auto first, int ka, int kw, bool wait) {
        const int w0 = uw + woff + fbase[1], a0 = ua + aoff + fbase[1];
        step(integral_constant<int, 0>{}, first, [&](auto mc) {
            constexpr int m = decltype(mc)::value;
            if constexpr (m < NR && m % 2 == 0) read(integral_constant<int, 1>{}, integral_constant<int, m / 2>{}, w0, a0);
            if constexpr (m >= NR && m % A_GAP == 0 && !(ABL & 4)) load_a((m - NR) / A_GAP, uf, ka);
        });
        MOE_LGKM0();
        if (wait) MOE_VMCNT(RING5 ? TM : TM + TN);
        MOE_BAR();
        const int w1 = uw1 + woff + fbase[0], a1 = ua1 + aoff + fbase[0];
        const int wdst = RING5 ? ua : uw;
        step(integral_constant<int, 1>{}, std::false_type{}, [&](auto mc) {
            constexpr int m = decltype(mc)::value;
            if constexpr (m < NR && m % 2 == 0) read(integral_constant<int, 0>{}, integral_constant<int, m / 2>{}, w1, a1);
            if constexpr (m < 4 * TN && m % 4 == 1 && !(ABL & 4)) load_w(m / 4, wdst, kw);
        });
        const int na1 = uf, nw1 = RING5 ? ua : uf + A_UNIT, nf = RING5 ? uw : ua;
        ua = ua1;
        uw = uw1;
        ua1 = na1;
        uw1 = nw1;
        uf = nf;
    };

    constexpr int W_AHEAD = RING5 ? 2 : 3;
    const int div = row_src != nullptr ? row_div : 1, packed = row_src != nullptr ? 0 : 1;
    bool fresh = true;
    for (;;) {
        b += stride;
        const WorkItem later = next.expert >= 0 ? item_at(b + stride) : next;
        int source = 0;
        if (row_src != nullptr && later.expert >= 0) source = *source_at(later);
        stage(std::true_type{}, 2, W_AHEAD, fresh);     // (behind an epilogue: see landed)
        for (int kt = 1; kt < KT; ++kt) {
            if (kt == KT - W_AHEAD) rsw = weights_of(next);
            if (kt == KT - 2) {
                rsa = rows_of(next);
#pragma unroll
                for (int q = 0; q < TM; ++q) a_src[q] = a_next[q];
            }
            const int ka = kt + 2, kw = kt + W_AHEAD;
            stage(std::false_type{}, ka < KT ? ka : ka - KT, kw < KT ? kw : kw - KT, true);
        }
        const auto ahead = prepare(item, wn, oct);
        MOE_MATRIX_RESULTS();
        // From here to the last accumulator's use there is no branch: values that cross one leave the AGPRs all at
        // once.  (And no read of an accumulator goes in front of the no-ops.)
        if constexpr (!(ABL & 1)) {
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int j = 0; j < TM; ++j) asm volatile("" : "+a"(acc[i][j]));
        }
        int here = lane;               // (so that the epilogue's addresses are not kept through the stages)
        asm volatile("" : "+v"(here));
        const W4Place<BM> place{lds + (RING5 ? uf : 3 * (A_UNIT + W_UNIT)) + wave * (W4Place<BM>::UR * 256), here, wm, wn,
                                here & 15, here >> 4};
        epilogue(acc, ahead, item, place, [&]() {
            MOE_SB();
            MOE_VMCNT(RING5 ? 0 : TN);            // the next tile's first two stages
            MOE_SB();
            int row = (source + own_row * packed) / div;
            asm volatile("" : "+v"(row));         // (a division that the compiler would jump over)
            a_offsets(row | (own_row < later.row1 - later.row0 ? 0 : -1), a_next);
            MOE_SB();
        });
        if (next.expert < 0) break;
        item = next;
        next = later;
        fresh = false;
    }
    MOE_VMCNT(0);
}
