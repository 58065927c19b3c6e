// Backward-filter for layers with few input channels (the 11x11 stride-4 first layer): a work-group keeps the whole
// K x (C*R*S) result in registers and walks the output rows of its share of the images with the input rows staged in
// LDS.  Two kernels: bf16 tensors on the bf16 matrix instruction (stride 4, pad 2; below) and fp32 tensors on the
// fp32 matrix instruction (second half of the file).
// Part of convnet_hotpath.hip: included there, inside its anonymous namespace, after conv_bf16_dma_kernels.h.
//
// --- bf16 ---
// GEMM view: dw[k][(c, r, s)] = sum over (n, p, q) of dy[n][k][p][q] * x[n][c][4p + r - 2][4q + s - 2], fp32 sums.
// v_mfma_f32_32x32x16_bf16 wants, per lane, eight CONSECUTIVE reduction indices of one row (one column) in a
// register quad.  The reduction runs along q inside one output row p (at most 64 positions, processed as
// 16-position blocks, zero beyond Q).  dy is contiguous along q; x is not (stride 4).  So every input row is
// staged in LDS once as S de-interleaved, shifted copies
//     E[c][row][s][q] = x[c][row - 2][4q + s - 2]            (zero outside the image, q = 0..63)
// and the operand of tap (c, r, s) for output row p is E[c][4p + r][s][q0 .. q0 + 7]: sixteen aligned bytes.  An
// input row is built once and serves every (p, r) pair that reads it: the rows live in a ring of 16 per channel,
// and a step (one output row p) adds the four rows the next step needs while the matrix instructions run.
// Building a row costs ~4 v_perm_b32 and one 16-byte LDS store per 8 outputs; the rows of dy (arbitrary 2-byte
// alignment in memory) are read as 4-byte-aligned words and shifted into place with v_alignbit_b32.
//
// One work-group (four waves) per CU owns the whole 96 x 384 result for its share of (image, output-row range)
// units: 3 x 3 blocks of 32 x 32 per wave, 144 accumulator registers, no reduction over work-groups inside the
// kernel.  Each work-group writes one partial result; reduce_partials adds them in a fixed order.
// LDS rows are 144 bytes (64 positions + 16): the 16 lanes of a ds_read_b128 phase read 16 consecutive filters
// (pitch 144) or 16 consecutive taps (pitch 144 per s, S * 144 per r), which covers the 64 banks once for S = 11.
constexpr int kRowsPitch = 144;            // bytes of 64 positions in LDS plus padding
constexpr int kRowsM = 96;                 // filters per work-group (three 32-row blocks)
constexpr int kRowsRing = 16;              // staged input rows per channel
constexpr int kRowsCols = 384;             // taps per work-group (four waves x three 32-column blocks)
constexpr int kRowsABuf = kRowsM * kRowsPitch;
// LDS bytes behind E that idle lanes store to (lane L at L * 16 + s * kRowsPitch, s <= 10): the steady-state step has
// no branch around a store, so that matrix instructions, the staging arithmetic and the LDS stores can be interleaved
constexpr int kRowsTrash = 255 * 16 + 10 * kRowsPitch + 16;

struct WgradRowsArgs {
    const unsigned short *x, *dy;
    float *part;                 // [work-group][K][Kg]
    int N, C, H, W, K, R, S, P, Q, Kg;         // stride 4, pad 2
    int x_bs, y_bs;              // elements between images (every offset into x and dy fits 31 bits)
    int dy_elems;                // elements of dy that may be read: (N - 1) * y_bs + K * P * Q
    int splits, units;           // output-row ranges per image; units = N * splits
    int ng;                      // groups of 8 positions per output row: ceil(Q / 8)
    int nkb;                     // 16-position blocks per output row: ceil(Q / 16)
    int nnew;                    // input rows a step adds per channel: min(R, 4)
    FastDiv div_splits, div_ng;
};

typedef unsigned int u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

// mask of output word i (elements 2i, 2i + 1) of a group of eight of which the first nv are real
__device__ __forceinline__ unsigned rows_mask(int nv, int i)
{
    return (2 * i < nv ? 0x0000FFFFu : 0u) | (2 * i + 1 < nv ? 0xFFFF0000u : 0u);
}

// Copy s of eight positions from the window of six 16-byte pieces that starts at input column 32g - 8:
// position i of copy s is window element 4i + s + 6.
template <int S_>
__device__ __forceinline__ void rows_store_copy(const u32x4 (&win)[6], char *dst, const unsigned (&mask)[4])
{
    constexpr int o = (S_ + 6) >> 1;                                // word of element 0 of this copy
    constexpr unsigned sel = (S_ & 1) ? 0x07060302u : 0x05040100u;  // high or low halves of the two words
    u32x4 out;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const unsigned lo = win[(4 * j + o) >> 2][(4 * j + o) & 3], hi = win[(4 * j + 2 + o) >> 2][(4 * j + 2 + o) & 3];
        out[j] = __builtin_amdgcn_perm(hi, lo, sel) & mask[j];
    }
    *reinterpret_cast<u32x4 *>(dst + S_ * kRowsPitch) = out;
}

// FULL: S = 11 and Q in 49..64 (four 16-position blocks), the first layer's case: those two are compile-time, and
// the LDS stores of the next row sit between the matrix instructions.
template <bool FULL>
__global__ __launch_bounds__(256, 1) void wgrad_rows_bf16_kernel(const WgradRowsArgs p)
{
    extern __shared__ __attribute__((aligned(16))) float lds_fast[];
    char *const lds = reinterpret_cast<char *>(lds_fast);      // dy rows, buffer 0 | buffer 1 | E
    char *const E = lds + 2 * kRowsABuf;
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int S = FULL ? 11 : p.S, nkb = FULL ? 4 : p.nkb;
    const int erow = S * kRowsPitch;                           // one staged input row: S copies
    const int echan = kRowsRing * erow;
    const int lds_bytes = 2 * kRowsABuf + p.C * echan;

    // positions >= 8 * ng are never written again: zero once
    for (int o = tid * 16; o < lds_bytes; o += 256 * 16) *reinterpret_cast<u32x4 *>(lds + o) = u32x4{0u, 0u, 0u, 0u};

    // this lane's three taps: byte offset of (c, ring row 0, s) in E and the filter row r
    int tap_off[3], tap_r[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        const int j = 32 * (3 * wave + t) + l32;
        const int jj = j < p.Kg ? j : 0;                       // columns beyond the filter read tap 0, never stored
        const int c = jj / (p.R * S), rs = jj - c * (p.R * S);
        const int r = rs / S, s = rs - r * S;
        tap_off[t] = c * echan + s * kRowsPitch + half * 16;
        tap_r[t] = r;
    }

    // E building: one (input row, group of 8 positions) pair per lane: six 16-byte pieces of the
    // row in (the window: input columns 32g - 8 .. 32g + 39), S copies out.  Loads and their use are kept apart (a
    // row is loaded three steps before it is needed): a load always reads a valid address -- a piece outside the row
    // reads the row's first piece, a row outside the image reads row 0 -- and zeros are put in when the window is
    // consumed.  Only two words of a window can hold padding that a real position reads: word 3 (columns -2, -1, for
    // g = 0) and word 0 of the piece that starts at column W (columns W, W + 1); everything else outside the row
    // only feeds positions >= Q, which the position masks clear.  FULL uses that; the general variant clears whole
    // pieces.
    auto e_load = [&](u32x4 (&win)[6], const char *img, int c, int hh, int g, bool on) {
        const int h = hh - 2;
        const bool rok = on & ((unsigned)h < (unsigned)p.H);
        const unsigned rowb = (unsigned)((c * p.H + (rok ? h : 0)) * p.W) * 2u;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const int start = 32 * g - 8 + 8 * k;               // W is a multiple of 8: a piece is inside or outside
            const bool ok = (unsigned)start < (unsigned)p.W;
            win[k] = *reinterpret_cast<const u32x4 *>(img + (size_t)(rowb + (ok ? (unsigned)start * 2u : 0u)));
        }
    };
    // zeros for what lies outside the image; the position masks of the group
    auto e_prepare = [&](u32x4 (&win)[6], unsigned (&mask)[4], int hh, int g) {
        const bool rok = (unsigned)(hh - 2) < (unsigned)p.H;
        if (FULL) {
            if (g == 0) win[0][3] = 0u;
#pragma unroll
            for (int k = 1; k < 6; ++k)
                if (32 * g - 8 + 8 * k == p.W) win[k][0] = 0u;
        } else {
#pragma unroll
            for (int k = 0; k < 6; ++k)
                if (!((unsigned)(32 * g - 8 + 8 * k) < (unsigned)p.W)) win[k] = u32x4{0u, 0u, 0u, 0u};
        }
        const int nv = rok ? min(max(p.Q - 8 * g, 0), 8) : 0;  // a row outside the image: every position zero
#pragma unroll
        for (int i = 0; i < 4; ++i) mask[i] = rows_mask(nv, i);
    };
    auto e_dst = [&](int c, int hh, int g) { return E + c * echan + (hh & (kRowsRing - 1)) * erow + g * 16; };
    char *const trash = E + p.C * echan + tid * 16;
    auto e_copy = [&](auto s_c, const u32x4 (&win)[6], char *dst, const unsigned (&mask)[4]) {
        constexpr int S_ = decltype(s_c)::value;
        if (S_ < S) rows_store_copy<S_>(win, dst, mask);
    };
    auto e_store_all = [&](u32x4 (&win)[6], int c, int hh, int g) {
        unsigned mask[4];
        e_prepare(win, mask, hh, g);
        char *dst = e_dst(c, hh, g);
        e_copy(std::integral_constant<int, 0>{}, win, dst, mask); e_copy(std::integral_constant<int, 1>{}, win, dst, mask);
        e_copy(std::integral_constant<int, 2>{}, win, dst, mask); e_copy(std::integral_constant<int, 3>{}, win, dst, mask);
        e_copy(std::integral_constant<int, 4>{}, win, dst, mask); e_copy(std::integral_constant<int, 5>{}, win, dst, mask);
        e_copy(std::integral_constant<int, 6>{}, win, dst, mask); e_copy(std::integral_constant<int, 7>{}, win, dst, mask);
        e_copy(std::integral_constant<int, 8>{}, win, dst, mask); e_copy(std::integral_constant<int, 9>{}, win, dst, mask);
        e_copy(std::integral_constant<int, 10>{}, win, dst, mask);
    };
    // steady state: the nnew rows a step adds, per channel (c, i) and group g: fixed per lane
    // (eight lanes per row, lane g of them idle for g >= ng: the 16-byte LDS stores of eight consecutive lanes then
    // go to one row's 128 consecutive bytes and never meet a bank twice)
    const int e_g = tid & 7;
    const bool e_on = (tid >> 3) < p.C * p.nnew && e_g < p.ng;
    int e_c, e_i;
    {
        const int t = e_on ? tid >> 3 : 0;
        e_c = t / p.nnew;
        e_i = t - e_c * p.nnew;
    }

    // dy rows: item (filter m, group j of 8 positions), three per thread; rows beyond K repeat row K - 1 (their
    // sums are never stored)
    const int nitems = kRowsM * p.ng;
    int a_base[3], a_dst[3], a_nv[3];
#pragma unroll
    for (int u = 0; u < 3; ++u) {
        const int it = min(tid + 256 * u, nitems - 1);
        const int m = (int)fastdiv((uint32_t)it, p.div_ng), j = it - m * p.ng;
        a_base[u] = min(m, p.K - 1) * p.P * p.Q + 8 * j;
        a_dst[u] = m * kRowsPitch + j * 16;
        a_nv[u] = min(max(p.Q - 8 * j, 0), 8);
    }
    // Five 4-byte words from the even element at or below the item's first one.  Where those 20 bytes would pass
    // the end of the tensor (the last group of its last row) the load reads element 0 instead and the item is
    // fetched one element at a time when it is consumed.
    unsigned a_mask[3][4];
#pragma unroll
    for (int u = 0; u < 3; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) a_mask[u][i] = rows_mask(a_nv[u], i);
    const char *const dyb = reinterpret_cast<const char *>(p.dy);
    auto a_load = [&](unsigned (&d)[3][5], int n, int prow) {
        const int rowbase = n * p.y_bs + prow * p.Q;
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            const int oe = (rowbase + a_base[u]) & ~1;          // 4-byte aligned element
            const unsigned off = oe + 10 <= p.dy_elems ? (unsigned)oe * 2u : 0u;
            const u32x4_a4 v = *reinterpret_cast<const u32x4_a4 *>(dyb + (size_t)off);
            d[u][0] = v[0]; d[u][1] = v[1]; d[u][2] = v[2]; d[u][3] = v[3];
            d[u][4] = *reinterpret_cast<const unsigned *>(dyb + (size_t)off + 16);
        }
    };
    auto a_shift_store = [&](int u, const unsigned (&d)[5], int o, char *dst) {
        const unsigned sh = (unsigned)(o & 1) * 16;
        u32x4 out;
#pragma unroll
        for (int i = 0; i < 4; ++i) out[i] = __builtin_amdgcn_alignbit(d[i + 1], d[i], sh) & a_mask[u][i];
        *reinterpret_cast<u32x4 *>(dst) = out;
    };
    // no branch: a thread without an item u stores to the trash area; an item at the tensor's end stores what the
    // clamped load returned and is put right by a_fix_tail before the barrier
    auto a_store_fast = [&](int u, const unsigned (&d)[5], int n, int prow, int buf) {
        char *dst = tid + 256 * u < nitems ? lds + buf * kRowsABuf + a_dst[u] : trash;
        a_shift_store(u, d, n * p.y_bs + prow * p.Q + a_base[u], dst);
    };
    auto a_fix_tail = [&](int n, int prow, int buf) {
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            const int o = n * p.y_bs + prow * p.Q + a_base[u];
            const int oe = o & ~1;
            if (tid + 256 * u < nitems && oe + 10 > p.dy_elems) {   // elements past the end lie beyond Q: masked
                unsigned d[5];
#pragma unroll
                for (int i = 0; i < 5; ++i) {
                    const unsigned lo = p.dy[min(oe + 2 * i, p.dy_elems - 1)];
                    const unsigned hi = p.dy[min(oe + 2 * i + 1, p.dy_elems - 1)];
                    d[i] = lo | (hi << 16);
                }
                a_shift_store(u, d, o, lds + buf * kRowsABuf + a_dst[u]);
            }
        }
    };
    // rows whose items can reach the tensor's end (a superset; a_fix_tail tests each item)
    auto near_end = [&](int n, int prow) { return n == p.N - 1 && (p.P - prow) * p.Q <= 8 * p.ng + 12; };
    auto a_store_one = [&](int u, const unsigned (&d)[5], int n, int prow, int buf) {
        if (tid + 256 * u < nitems) a_store_fast(u, d, n, prow, buf);
    };

    f32x16 acc[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][t][v] = 0.f;

    // three register stages: stage (row - p_begin) % 3 holds the loads of that output row
    u32x4 win[3][6];
    unsigned dd[3][3][5];

    for (int unit = blockIdx.x; unit < p.units; unit += gridDim.x) {
        const int n = (int)fastdiv((uint32_t)unit, p.div_splits);
        const int sp = unit - n * p.splits;
        const int p_begin = (int)((int64_t)p.P * sp / p.splits), p_end = (int)((int64_t)p.P * (sp + 1) / p.splits);
        if (p_begin >= p_end) continue;
        __syncthreads();                                        // zero fill / the previous unit's reads are done
        const char *const img = reinterpret_cast<const char *>(p.x + (size_t)n * p.x_bs);
        auto issue = [&](auto st_c, int prow) {                 // loads of output row prow (clamped to the unit)
            constexpr int ST = decltype(st_c)::value;
            const int pr = min(prow, p_end - 1);
            e_load(win[ST], img, e_c, 4 * pr + p.R - p.nnew + e_i, e_g, e_on);
            a_load(dd[ST], n, pr);
        };
        // every input row of the first output row, and its dy rows
        {
            const int rows = p.C * p.R;
            for (int t0 = 0; t0 < rows; t0 += 32) {
                const int t1 = t0 + (tid >> 3), g = tid & 7;
                const bool on = t1 < rows && g < p.ng;
                const int t = on ? t1 : 0;
                const int c = t / p.R, i = t - c * p.R;
                e_load(win[0], img, c, 4 * p_begin + i, g, on);
                if (on) e_store_all(win[0], c, 4 * p_begin + i, g);
            }
            a_load(dd[0], n, p_begin);
#pragma unroll
            for (int u = 0; u < 3; ++u) a_store_one(u, dd[0][u], n, p_begin, 0);
            if (near_end(n, p_begin)) a_fix_tail(n, p_begin, 0);
        }
        issue(std::integral_constant<int, 1>{}, p_begin + 1);
        issue(std::integral_constant<int, 2>{}, p_begin + 2);
        __syncthreads();
        int buf = 0;
        // One output row: loads of row prow + 3 into the stage row prow used; matrix instructions of row prow; the
        // stage of row prow + 1 goes to LDS (dy buffer buf ^ 1, ring rows no tap of row prow reads).  After the last
        // row of the unit the stores repeat that row into places nothing reads before they are rewritten.
        auto step = [&](auto st_c, int prow) {
            constexpr int ST = decltype(st_c)::value, SN = (ST + 1) % 3;
            issue(st_c, prow + 3);
            const int pn = min(prow + 1, p_end - 1);            // the row stage SN holds
            const int hh_new = 4 * (prow + 1) + p.R - p.nnew + e_i;
            const char *Ab = lds + buf * kRowsABuf + l32 * kRowsPitch + half * 16;
            const char *Bb[3];
#pragma unroll
            for (int t = 0; t < 3; ++t) Bb[t] = E + tap_off[t] + ((4 * prow + tap_r[t]) & (kRowsRing - 1)) * erow;
            bf16x8 fa[2][3], fb[2][3];
            auto read = [&](int set, int kb) {
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    fa[set][i] = *reinterpret_cast<const bf16x8 *>(Ab + i * 32 * kRowsPitch + kb * 32);
#pragma unroll
                for (int t = 0; t < 3; ++t) fb[set][t] = *reinterpret_cast<const bf16x8 *>(Bb[t] + kb * 32);
            };
            unsigned mask[4];
            char *dst = e_on ? e_dst(e_c, hh_new, e_g) : trash;
            // store work in twelve slots: copy s of the new input rows in slot s, a dy item in slots 3, 7, 11.
            // FULL: no branches (idle lanes store to the trash area), so the whole step is one scheduling region
            auto slot = [&](auto k_c) {
                constexpr int K_ = decltype(k_c)::value;
                // (the four words of the window no copy reads stay allocated until here: the register allocator would
                // otherwise hand them out while their load is in flight, and every such reuse waits for the load)
                if (K_ == 0)
                    asm volatile("" :: "v"(win[SN][0][0]), "v"(win[SN][0][1]), "v"(win[SN][0][2]), "v"(win[SN][5][3]));
                if (FULL) {
                    if (K_ == 0) e_prepare(win[SN], mask, 4 * pn + p.R - p.nnew + e_i, e_g);
                    if (K_ < 11) e_copy(std::integral_constant<int, K_ < 11 ? K_ : 0>{}, win[SN], dst, mask);
                    if (K_ % 4 == 3) a_store_fast(K_ / 4, dd[SN][K_ / 4], n, pn, buf ^ 1);
                } else {
                    if (K_ == 0 && e_on) e_prepare(win[SN], mask, 4 * pn + p.R - p.nnew + e_i, e_g);
                    if (K_ < 11 && e_on) e_copy(std::integral_constant<int, K_ < 11 ? K_ : 0>{}, win[SN], dst, mask);
                    if (K_ % 4 == 3) a_store_one(K_ / 4, dd[SN][K_ / 4], n, pn, buf ^ 1);
                }
            };
            read(0, 0);
            if (FULL) {
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) {
                    if (kb + 1 < 4) read((kb + 1) & 1, kb + 1);
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
#pragma unroll
                        for (int t = 0; t < 3; ++t)
                            acc[i][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kb & 1][i], fb[kb & 1][t], acc[i][t],
                                                                                0, 0, 0);
                        if (kb == 0) { if (i == 0) slot(std::integral_constant<int, 0>{}); if (i == 1) slot(std::integral_constant<int, 1>{}); if (i == 2) slot(std::integral_constant<int, 2>{}); }
                        if (kb == 1) { if (i == 0) slot(std::integral_constant<int, 3>{}); if (i == 1) slot(std::integral_constant<int, 4>{}); if (i == 2) slot(std::integral_constant<int, 5>{}); }
                        if (kb == 2) { if (i == 0) slot(std::integral_constant<int, 6>{}); if (i == 1) slot(std::integral_constant<int, 7>{}); if (i == 2) slot(std::integral_constant<int, 8>{}); }
                        if (kb == 3) { if (i == 0) slot(std::integral_constant<int, 9>{}); if (i == 1) slot(std::integral_constant<int, 10>{}); if (i == 2) slot(std::integral_constant<int, 11>{}); }
                    }
                }
                // A wave issues in order: while it waits to issue the next matrix instruction nothing else of it
                // issues.  So one matrix instruction (32 clocks in its pipe) is followed by up to seven vector
                // instructions (4 clocks each) and one LDS / memory instruction, 36 times.
                // The fragments of the next 16 positions are read in one go before the nine instructions that
                // hide their latency.
                __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);          // LDS reads: fragments of block 0
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) {
                    if (kb < 3) __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
                    for (int g = 0; g < 9; ++g) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // matrix
                        __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);  // vector ALU
                        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);  // LDS write
                    }
                }
                if (near_end(n, pn)) a_fix_tail(n, pn, buf ^ 1);
            } else {
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) {
                    if (kb < nkb) {
                        if (kb + 1 < nkb) read((kb + 1) & 1, kb + 1);
#pragma unroll
                        for (int i = 0; i < 3; ++i)
#pragma unroll
                            for (int t = 0; t < 3; ++t)
                                acc[i][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kb & 1][i], fb[kb & 1][t],
                                                                                    acc[i][t], 0, 0, 0);
                    }
                }
                slot(std::integral_constant<int, 0>{}); slot(std::integral_constant<int, 1>{});
                slot(std::integral_constant<int, 2>{}); slot(std::integral_constant<int, 3>{});
                slot(std::integral_constant<int, 4>{}); slot(std::integral_constant<int, 5>{});
                slot(std::integral_constant<int, 6>{}); slot(std::integral_constant<int, 7>{});
                slot(std::integral_constant<int, 8>{}); slot(std::integral_constant<int, 9>{});
                slot(std::integral_constant<int, 10>{}); slot(std::integral_constant<int, 11>{});
                if (near_end(n, pn)) a_fix_tail(n, pn, buf ^ 1);
            }
            __syncthreads();
            buf ^= 1;
        };
        // (no way out of the loop between its three steps: an edge from there back to the loop head would carry
        // loads that were just issued, and the first register reuse at the head would wait for them)
        int prow = p_begin;
        for (; prow + 3 <= p_end; prow += 3) {
            step(std::integral_constant<int, 0>{}, prow);
            step(std::integral_constant<int, 1>{}, prow + 1);
            step(std::integral_constant<int, 2>{}, prow + 2);
        }
        if (prow < p_end) step(std::integral_constant<int, 0>{}, prow);
        if (prow + 1 < p_end) step(std::integral_constant<int, 1>{}, prow + 1);
    }

    float *out = p.part + (size_t)blockIdx.x * p.K * p.Kg;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            const int col = 32 * (3 * wave + t) + l32;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = 32 * i + (v >> 2) * 8 + half * 4 + (v & 3);
                if (row < p.K && col < p.Kg) out[(size_t)row * p.Kg + col] = acc[i][t][v];
            }
        }
}

// ---------------------------------------------------------------------------
// The same decomposition for fp32 tensors (v_mfma_f32_32x32x2_f32: one value per lane and operand, so no
// alignment question and no shifted copies): a work-group owns the whole K x (C*R*S) result for its (image,
// output-row range) units and walks the output rows.  Twelve waves, three per SIMD -- a wave that waits for its
// LDS reads or at the barrier leaves the matrix pipe to the other two --, each with the 96 rows x 32 taps of one
// column block in registers (3 blocks of 32 x 32).  Per output row p the LDS holds
//   xr[c][ring row][WP]   the input rows stride*p .. (fp32, zero padding columns in place, ring of 16 rows per
//                         channel; a step adds the `stride` rows the next output row needs)
//   dyr[buf][m][58]       dy(n, m, p, 0..Q-1), zero from Q on; pitch 58: the 64 lanes (m, k parity) of one read
//                         cover the 64 banks once
// and reduction pair t (positions 2t, 2t+1) costs four single-word LDS reads per wave -- three dy values, one
// input value at patch offset row*WP + stride*(2t + k) + s -- for three matrix instructions of 64 clocks, all
// with immediate offsets.  One output row is 9 * ceil(Q/2) matrix instructions per SIMD (16 k clocks for the
// first layer) against a few hundred clocks of staging, so the next row's loads simply sit in registers across
// the row.
// ---------------------------------------------------------------------------
constexpr int kRowsF32Threads = 768;
constexpr int kRowsF32DyPitch = 58;
constexpr int kRowsF32DyBuf = kRowsM * kRowsF32DyPitch;       // floats per dy buffer
constexpr int kRowsF32Slack = 64;                             // floats behind the input rows: reads one pair too far

struct WgradRowsF32Args {
    const float *x, *dy;
    float *part;                 // [work-group][K][Kg]
    int N, C, H, W, K, R, S, P, Q, Kg, stride, pad;
    int x_bs, y_bs;
    int splits, units;
    int WP;                      // LDS row pitch in floats: >= W + 2 * pad, = 48 mod 64
    int nnew;                    // input rows a step adds per channel: min(R, stride)
    FastDiv div_splits;
};

__global__ __launch_bounds__(kRowsF32Threads, 1) void wgrad_rows_f32_kernel(const WgradRowsF32Args p)
{
    extern __shared__ __attribute__((aligned(16))) float lds_fast[];
    float *const dyr = lds_fast;                               // two buffers
    float *const xr = lds_fast + 2 * kRowsF32DyBuf;
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int xchan = kRowsRing * p.WP;
    const int lds_floats = 2 * kRowsF32DyBuf + p.C * xchan + kRowsF32Slack;
    for (int o = tid; o < lds_floats; o += kRowsF32Threads) lds_fast[o] = 0.f;   // padding, positions >= Q: zero

    // this lane's tap: float offset of (c, ring row 0, column s + stride * k parity) and the filter row r
    int tap_off, tap_r;
    {
        const int j = 32 * wave + l32;
        const int jj = j < p.Kg ? j : 0;
        const int c = jj / (p.R * p.S), rs = jj - c * (p.R * p.S);
        const int r = rs / p.S, s = rs - r * p.S;
        tap_off = c * xchan + s + p.stride * half;
        tap_r = r;
    }

    f32x16 acc[3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;

    // Staging with addresses that cost nothing per element: thread t owns position q = t % 64 of the dy rows
    // m = t / 64 + 12u (u = 0..7) and column w = t % 256 of the new input rows (c, i) = slot t / 256 + 3v
    // (v = 0..5, slot = 4c + i); what changes from element to element is uniform.
    constexpr int NDY = kRowsM / 12;                           // 8 dy values per thread
    constexpr int NXR = 6;
    const int dq = tid & 63, dm = tid >> 6;
    const bool dq_on = dq < p.Q;
    const int xw = tid & 255, xs0 = tid >> 8;
    const int nfull = p.Q >> 1;                                // reduction pairs with both positions

    for (int unit = blockIdx.x; unit < p.units; unit += gridDim.x) {
        const int n = (int)fastdiv((uint32_t)unit, p.div_splits);
        const int sp = unit - n * p.splits;
        const int p_begin = (int)((int64_t)p.P * sp / p.splits), p_end = (int)((int64_t)p.P * (sp + 1) / p.splits);
        if (p_begin >= p_end) continue;
        const float *xn = p.x + (size_t)n * p.x_bs, *dyn = p.dy + (size_t)n * p.y_bs;
        __syncthreads();
        // input rows first_hh .. first_hh + rows - 1 (image row = hh - pad) of every channel; rows outside the
        // image are zero.  (Loads read a clamped, always valid address and nothing touches the value before the
        // matching store: a select on a loaded value would make the thread wait for each load in turn.)
        auto load_x = [&](float (&v)[NXR], int first_hh, int rows) {
            const int w = min(xw, p.W - 1);
#pragma unroll
            for (int u = 0; u < NXR; ++u) {
                const int slot = xs0 + 3 * u, c = slot >> 2, i = slot & 3;
                const int h = min(max(first_hh + i - p.pad, 0), p.H - 1);
                v[u] = xn[(min(c, p.C - 1) * p.H + h) * p.W + w];
            }
        };
        auto store_x = [&](const float (&v)[NXR], int first_hh, int rows) {
#pragma unroll
            for (int u = 0; u < NXR; ++u) {
                const int slot = xs0 + 3 * u, c = slot >> 2, i = slot & 3;
                if (c < p.C && i < rows && xw < p.W) {
                    const bool inside = (unsigned)(first_hh + i - p.pad) < (unsigned)p.H;
                    xr[c * xchan + ((first_hh + i) & (kRowsRing - 1)) * p.WP + p.pad + xw] = inside ? v[u] : 0.f;
                }
            }
        };
        auto load_dy = [&](float (&v)[NDY], int prow) {
            const float *src = dyn + prow * p.Q + min(dq, p.Q - 1);
#pragma unroll
            for (int u = 0; u < NDY; ++u) v[u] = src[min(dm + 12 * u, p.K - 1) * p.P * p.Q];
        };
        auto store_dy = [&](const float (&v)[NDY], int buf) {
            float *dst = dyr + buf * kRowsF32DyBuf + dm * kRowsF32DyPitch + dq;
            if (dq_on) {
#pragma unroll
                for (int u = 0; u < NDY; ++u)
                    if (dm + 12 * u < p.K) dst[12 * u * kRowsF32DyPitch] = v[u];
            }
        };
        float vx[NXR], vdy[NDY];
        // every input row of the first output row (R rows, in passes of nnew), and its dy row
        for (int r0 = 0; r0 < p.R; r0 += p.nnew) {
            const int rows = min(p.nnew, p.R - r0);
            load_x(vx, p.stride * p_begin + r0, rows);
            store_x(vx, p.stride * p_begin + r0, rows);
        }
        load_dy(vdy, p_begin);
        store_dy(vdy, 0);
        __syncthreads();
        int buf = 0;
        for (int prow = p_begin; prow < p_end; ++prow) {
            const bool more = prow + 1 < p_end;
            const int hh_new = p.stride * (prow + 1) + p.R - p.nnew;
            if (more) {
                load_x(vx, hh_new, p.nnew);
                load_dy(vdy, prow + 1);
            }
            const float *Ab = dyr + buf * kRowsF32DyBuf + l32 * kRowsF32DyPitch + half;
            const float *Bb = xr + tap_off + ((p.stride * prow + tap_r) & (kRowsRing - 1)) * p.WP;
            float fa[2][3], fb[2];
            // operands of pair tp; a pair past the last one may be read (never used): the reads stay inside LDS
            auto read = [&](int set, int tp) {
#pragma unroll
                for (int i = 0; i < 3; ++i) fa[set][i] = Ab[i * 32 * kRowsF32DyPitch + 2 * tp];
                fb[set] = Bb[2 * p.stride * tp];
            };
            auto mfmas = [&](int set) {
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[set][i], fb[set], acc[i], 0, 0, 0);
            };
            read(0, 0);
            int tp = 0;
            // no branch inside (the waits count the reads), and the order is pinned: the reads of the next pair
            // are issued before this pair's matrix instructions
            for (; tp + 2 <= nfull; tp += 2) {
                read(1, tp + 1);
                __builtin_amdgcn_sched_barrier(0);
                mfmas(0);
                __builtin_amdgcn_sched_barrier(0);
                read(0, tp + 2);
                __builtin_amdgcn_sched_barrier(0);
                mfmas(1);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (tp < nfull) {                                   // set 0 holds pair tp
                if (p.Q & 1) read(1, tp + 1);
                mfmas(0);
                ++tp;
                if (p.Q & 1) {
                    // last position alone: the missing odd position reads dy's zero at Q and, for the input, that
                    // same zero word, so that no input value is multiplied by it
                    if (half) fb[1] = fa[1][0];
                    mfmas(1);
                }
            } else if (p.Q & 1) {                               // set 0 holds the half pair nfull
                if (half) fb[0] = fa[0][0];
                mfmas(0);
            }
            if (more) {
                store_x(vx, hh_new, p.nnew);
                store_dy(vdy, buf ^ 1);
            }
            __syncthreads();
            buf ^= 1;
        }
    }

    float *out = p.part + (size_t)blockIdx.x * p.K * p.Kg;
    const int col = 32 * wave + l32;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = 32 * i + (v >> 2) * 8 + half * 4 + (v & 3);
            if (row < p.K && col < p.Kg) out[(size_t)row * p.Kg + col] = acc[i][v];
        }
}

// ---------------------------------------------------------------------------
// fp32 tensors on the bf16 matrix instruction, operands split into three bfloat16 parts (six products, two accumulators:
// arithmetic, error and range as in conv_split_kernels.h), for stride 4.  The same decomposition: a work-group owns the whole
// K x (C*R*S) result for its (image, output-row range) units.
//
// Columns come in quads, four consecutive taps s = 4 sg .. 4 sg + 3 of one (c, r): at output column q they are the input
// columns 4 (q + sg) .. + 3 of the padded row, eight aligned bytes of a staged part.  That is the piece that
// ds_read_b64_tr_b16 takes from a lane, so the transposed operand (eight consecutive q of a tap per lane) comes straight from
// the input row as it lies in memory: no shifted copies, which in three parts would not fit the LDS.  S = 11 costs one unused
// column in twelve.
//   dy   [buffer][part][96 filters][144 bytes]: 64 positions, zero from Q on
//   x    [c][ring row]: three parts of 456 bytes, padded input columns 0 .. 4 Q + 7, and 72 bytes of zeros; 1440 = 160 mod 256
//        keeps the filter rows that a read meets in different banks
// The result is 3 x 13 blocks of 32 x 32, five to each of eight waves (two per SIMD, so that one's splitting and LDS stores
// pass under the other's matrix instructions): the three rows of column block `wave`, and two of the fifteen blocks of
// columns 8..12 (rows_split_extra).  An output row is 4 x 30 matrix instructions per wave; the next row's values are loaded at
// its start and split and stored between its 16-position blocks.
// From position Q on dy is zero and the input holds values of other windows of the same row, or zeros: where one of those is
// not finite the sum becomes NaN, and the rule below computes it again unless a NaN of its own explains it.
// Bound: matrix instructions (128 x 3 x 224 x 224, 96 filters 11 x 11: 30 x 110 x 32 clocks x 2 waves = 106 us at 2 GHz).
// Measured: that layer's calls (forward and this) 488 -> 397 us; kernel in the running network 267 -> 175 us; matrix unit busy
// 64 % of the cycles in which a CU holds work-groups, 55 % of the duration; error against 64 bits 7.0e-7 -> 2.6e-7.  What was costly on the way: bounds and indexes worked out at each
// load (506 vector instructions per wave and row, 214 now), masks on the operand of the last block, and sums that spilled.
// ---------------------------------------------------------------------------
constexpr int kRowsSplitDyPart = kRowsM * kRowsPitch;
constexpr int kRowsSplitDyBuf = 3 * kRowsSplitDyPart;
// What a row's reads reach past a part is another part of the same row or the zeros behind them, never a row that is being staged.
static_assert(2 * kRowsSplitPitch + rows_split_read_end(4) <= kRowsSplitRow, "reads stay inside their row");
static_assert(kRowsSplitRow % 16 == 0, "cleared 16 bytes at a time");

struct WgradRowsSplitArgs {
    const float *x, *dy;
    float *part;                 // [work-group][K][Kg]
    int C, H, W, K, R, S, P, Q, Kg, pad;       // stride 4
    int x_bs, y_bs;              // elements between images
    unsigned x_bytes, dy_bytes;  // from the first element to the last
    int splits, units;
    int SG, quads;               // ceil(S / 4); C * R * SG <= 104
    int nnew;                    // input rows a step adds per channel: min(R, 4)
    int xg, dyg;                 // groups of four: padded input columns, output columns
    FastDiv div_splits, div_xg, div_dyg, div_nnew;
};

// Blocks of column blocks 8..12 that a wave computes beside its own: (row block, column block) twice, the row blocks different.
// The last of the sixteen repeats a block, which is not stored.
struct RowsSplitExtra { int row0, col0, row1, col1; };
__device__ __forceinline__ RowsSplitExtra rows_split_extra(int wave)
{
    constexpr unsigned table[8] = {0x0818, 0x1929, 0x2A0A, 0x091A, 0x0B1B, 0x1C2C, 0x2B0C, 0x280F};
    const unsigned t = table[wave & 7];
    return RowsSplitExtra{(int)(t >> 12), (int)(t >> 8 & 15), (int)(t >> 4 & 15), (int)(t & 15)};
}

// NKB: blocks of 16 positions per output row
template <int NKB>
__global__ __launch_bounds__(kRowsSplitThreads, 1) void wgrad_rows_split_kernel(const WgradRowsSplitArgs p)
{
    constexpr unsigned kOutside = 0x80000000u;
    constexpr int NW = kRowsSplitThreads / 64;
    extern __shared__ __attribute__((aligned(16))) float lds_fast[];
    char *const lds = reinterpret_cast<char *>(lds_fast);
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const int echan = kRowsRing * kRowsSplitRow;

    // zero: dy's positions from Q on, and whatever the input's positions from there on may read before it is staged
    for (int o = tid * 16; o < 2 * kRowsSplitDyBuf + p.C * echan; o += kRowsSplitThreads * 16)
        *reinterpret_cast<u32x4 *>(lds + o) = u32x4{0u, 0u, 0u, 0u};

    const auto rsrc_x = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.x), 0, (int)p.x_bytes, 0x00020000);
    const auto rsrc_dy = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.dy), 0, (int)p.dy_bytes, 0x00020000);

    // row blocks in the order slot 0, 1 (which serve the two extra blocks), 2; column blocks: own, of slot 0, of slot 1
    const RowsSplitExtra ex = rows_split_extra(wave);
    const int slot_row[3] = {ex.row0, ex.row1, 3 - ex.row0 - ex.row1};
    const int blk_col[3] = {wave, ex.col0, min(ex.col1, 12)};
    const bool stored4 = ex.col1 < 13;

    // this lane's address in a column block, position (lane % 16) / 4 of its half and quad lane % 4 of sixteen columns, and
    // the quad's filter row from bit 24 on
    unsigned tap[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const int quad = blk_col[b] * 8 + ((lane >> 4) & 1) * 4 + (lane & 3);
        const int qq = quad < p.quads ? quad : 0;                 // quads past the last: computed, never stored
        const int cr = qq / p.SG, sg = qq - cr * p.SG;
        const int c = cr / p.R;
        tap[b] = (unsigned)(2 * kRowsSplitDyBuf + c * echan + (half * 8 + ((lane & 15) >> 2) + sg) * 8) |
                 (unsigned)(cr - c * p.R) << 24;
    }

    f32x16 acc[5], low[5];
#pragma unroll
    for (int t = 0; t < 5; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) { acc[t][v] = 0.f; low[t][v] = 0.f; }

    // Staging items of four values: two of x (c, new row i, group of padded columns) and three of dy (filter, group of
    // positions) per thread.  Kept per item: byte offset in its tensor from the row of an output row on (kOutside: no item),
    // byte offset in LDS (of x: of ring row 0, i from bit 24 on), and four bits that say which values are inside the row.
    unsigned x_off[2], x_lds[2], dy_off[3], dy_lds[3], inside = 0;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int it = tid + kRowsSplitThreads * u;
        const int t = (int)fastdiv((uint32_t)it, p.div_xg), g = it - t * p.xg;
        const int c = (int)fastdiv((uint32_t)t, p.div_nnew), i = t - c * p.nnew, w = 4 * g - p.pad;
        x_off[u] = c < p.C ? (unsigned)((c * p.H + i) * p.W + w) * 4u : kOutside;
        x_lds[u] = c < p.C ? (unsigned)(2 * kRowsSplitDyBuf + c * echan + g * 8) | (unsigned)i << 24 : kOutside;
#pragma unroll
        for (int e = 0; e < 4; ++e) inside |= (unsigned)(w + e) < (unsigned)p.W ? 1u << (4 * u + e) : 0u;
    }
#pragma unroll
    for (int u = 0; u < 3; ++u) {
        const int it = tid + kRowsSplitThreads * u;
        const int m = (int)fastdiv((uint32_t)it, p.div_dyg), g = it - m * p.dyg;
        dy_off[u] = m < p.K ? (unsigned)(m * p.P * p.Q + 4 * g) * 4u : kOutside;
        dy_lds[u] = m < p.K ? (unsigned)(m * kRowsPitch + g * 8) : kOutside;
#pragma unroll
        for (int e = 0; e < 4; ++e) inside |= 4 * g + e < p.Q ? 1u << (8 + 4 * u + e) : 0u;
    }
    // rows outside the image read as zero; a row past the unit's last one reads what is there and is not used
    auto load_x = [&](float (&v)[4], int u, int n, int first_hh) {
        const int h0 = first_hh - p.pad;
        const bool ok = (unsigned)(h0 + (int)(x_lds[u] >> 24)) < (unsigned)p.H;       // (no item: row 128 and up)
        const unsigned base = x_off[u] + (unsigned)(n * p.x_bs + h0 * p.W) * 4u;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            v[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc_x, ok ? base + 4u * e : kOutside, 0, 0));
    };
    auto load_dy = [&](float (&v)[4], int u, int n, int prow) {
        const unsigned base = dy_off[u] + (unsigned)(n * p.y_bs + prow * p.Q) * 4u;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            v[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc_dy, base + 4u * e, 0, 0));
    };
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    u32x2 sp[3];
    auto split_two = [&](const float (&v)[4], int t, int bit) {   // values 2t, 2t + 1 of the item whose bits start at `bit`
        auto in = [&](int e) {
            return __uint_as_float(__float_as_uint(v[e]) & (unsigned)__builtin_amdgcn_sbfe((int)inside, bit + e, 1));
        };
        unsigned h, m, l;
        split_pair(in(2 * t), in(2 * t + 1), h, m, l);
        sp[0][t] = h; sp[1][t] = m; sp[2][t] = l;
    };
    auto put = [&](char *dst, int part_bytes) {
#pragma unroll
        for (int c = 0; c < 3; ++c) *reinterpret_cast<u32x2 *>(dst + c * part_bytes) = sp[c];
    };
    auto put_x = [&](int u, int first_hh, int rows) {
        const int i = (int)x_lds[u] >> 24;
        if ((i >= 0) & (i < rows))
            put(lds + (x_lds[u] & 0xffffffu) + ((unsigned)(first_hh + i) & (kRowsRing - 1)) * kRowsSplitRow, kRowsSplitPitch);
    };
    auto store_x = [&](const float (&v)[4], int u, int first_hh, int rows) {
        split_two(v, 0, 4 * u); split_two(v, 1, 4 * u);
        put_x(u, first_hh, rows);
    };
    auto put_dy = [&](int u, int buf) {
        if ((int)dy_lds[u] >= 0) put(lds + buf * kRowsSplitDyBuf + dy_lds[u], kRowsSplitDyPart);
    };
    auto store_dy = [&](const float (&v)[4], int u, int buf) {
        split_two(v, 0, 8 + 4 * u); split_two(v, 1, 8 + 4 * u);
        put_dy(u, buf);
    };

    typedef __attribute__((address_space(3))) char *lds_bytes;
    typedef __attribute__((address_space(3))) s16x4 *lds_quad;
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    s16x8 fa[2][3], fb[2][3];                                     // [set][part]
    unsigned a_off[3], b_off[3];
    auto read_a = [&](int set, int slot, int kb) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
            fa[set][c] = *reinterpret_cast<const s16x8 *>(lds + a_off[slot] + c * kRowsSplitDyPart + kb * 32);
    };
    auto read_b = [&](int set, int b, int kb) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const lds_bytes a = (lds_bytes)lds + b_off[b] + c * kRowsSplitPitch + kb * 128;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad)a);
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad)(a + 32));
            fb[set][c] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
    };
    auto product = [&](int tile, int a, int b, int ca, int cb) {
        f32x16 &sum = ca + cb == 0 ? acc[tile] : low[tile];
        sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa[a][ca]),
                                                      __builtin_bit_cast(bf16x8, fb[b][cb]), sum, 0, 0, 0);
    };

    for (int unit = blockIdx.x; unit < p.units; unit += gridDim.x) {
        const int n = (int)fastdiv((uint32_t)unit, p.div_splits);
        const int sp = unit - n * p.splits;
        const int p_begin = (int)((int64_t)p.P * sp / p.splits), p_end = (int)((int64_t)p.P * (sp + 1) / p.splits);
        if (p_begin >= p_end) continue;
        __syncthreads();                                          // zero fill / the previous unit's reads are done
        {
            float d0[4], d1[4], d2[4], x0[4], x1[4];
            load_dy(d0, 0, n, p_begin); load_dy(d1, 1, n, p_begin); load_dy(d2, 2, n, p_begin);
#pragma unroll 1
            for (int r0 = 0; r0 < p.R; r0 += p.nnew) {            // every input row of the first output row
                const int hh = 4 * p_begin + r0, rows = min(p.nnew, p.R - r0);
                load_x(x0, 0, n, hh); load_x(x1, 1, n, hh);
                store_x(x0, 0, hh, rows); store_x(x1, 1, hh, rows);
            }
            store_dy(d0, 0, 0); store_dy(d1, 1, 0); store_dy(d2, 2, 0);
        }
        __syncthreads();
        int buf = 0;
        for (int prow = p_begin; prow < p_end; ++prow) {
            const int hh_new = 4 * (prow + 1) + p.R - p.nnew;
#pragma unroll
            for (int i = 0; i < 3; ++i)
                a_off[i] = (unsigned)(buf * kRowsSplitDyBuf + (slot_row[i] * 32 + l32) * kRowsPitch + half * 16);
#pragma unroll
            for (int b = 0; b < 3; ++b)
                b_off[b] = (tap[b] & 0xffffffu) + ((4u * prow + (tap[b] >> 24)) & (kRowsRing - 1)) * kRowsSplitRow;
            read_b(0, 0, 0);
            read_a(0, 2, 0);
            __builtin_amdgcn_sched_barrier(0);
            float v0[4], v1[4], v2[4];                            // values of the next row: two items of dy, then the others
            load_dy(v0, 0, n, prow + 1); load_dy(v1, 1, n, prow + 1);
            __builtin_amdgcn_sched_barrier(0);
            // One block of 16 positions.  The filters' fragments of a slot alternate between two sets, the own column block stays
            // in set 0 of the inputs and the extra ones pass through set 1: 48 registers of operands beside 160 of sums.  The
            // next row's values are split and stored between matrix instructions, one pair of a thread's four at a time: dy's
            // first two items in block 1, the others, loaded at the end of that block, in the last.  Rows of fewer than four blocks
            // take the first two in the last block and the others after it: closer together they do not fit the registers
            // (three blocks: 66 spills in the loop, 608 us where rows of 55 positions take 160).  Past the unit's last row
            // that writes where nothing is read.
            constexpr int KA = NKB > 3 ? 1 : NKB - 1, KB = NKB > 3 ? NKB - 1 : NKB;
            auto work = [&](auto kb_c, auto m_c) {
                constexpr int kb = decltype(kb_c)::value, i = decltype(m_c)::value - (kb == KA ? 20 : 16);
                if constexpr ((kb == KA || kb == KB) && i >= 0) {
                    constexpr int u = i / 3, s = i % 3;
                    if constexpr (kb == KA && u < 2) {
                        if constexpr (s < 2) split_two(u == 0 ? v0 : v1, s, 8 + 4 * u); else put_dy(u, buf ^ 1);
                    } else if constexpr (kb == KB && u < 3) {
                        if constexpr (s < 2) split_two(u == 0 ? v0 : u == 1 ? v1 : v2, s, u == 0 ? 16 : 4 * (u - 1));
                        else if constexpr (u == 0) put_dy(2, buf ^ 1);
                        else put_x(u - 1, hh_new, p.nnew);
                    }
                }
            };
            auto second_loads = [&]() {
                load_dy(v0, 2, n, prow + 1); load_x(v1, 0, n, hh_new); load_x(v2, 1, n, hh_new);
            };
            auto block = [&](auto kb_c) {
                constexpr int kb = decltype(kb_c)::value, U = kb & 1, V = U ^ 1;
                constexpr bool last = kb + 1 == NKB;
                static_for<30>([&](auto m_c) {
                    constexpr int m = decltype(m_c)::value;
                    if constexpr (m == 0) { read_a(V, 0, kb); read_b(1, 1, kb); }
                    if constexpr (m == 6) read_a(U, 1, kb);
                    if constexpr (m == 18) read_b(1, 2, kb);
                    if constexpr (m == 24 && !last) { read_b(0, 0, kb + 1); read_a(V, 2, kb + 1); }
                    __builtin_amdgcn_sched_barrier(0);
                    constexpr int ca[6] = {2, 0, 0, 1, 0, 1}, cb[6] = {0, 0, 2, 0, 1, 1};
                    constexpr int g = m < 6 ? m : m < 18 ? (m - 6) / 2 : m < 24 ? m - 18 : m - 24;
                    constexpr int tile = m < 6 ? 2 : m < 18 ? (m & 1) * 3 : m < 24 ? 1 : 4;
                    product(tile, m < 6 || m >= 18 ? U : V, tile < 3 ? 0 : 1, ca[g], cb[g]);
                    __builtin_amdgcn_sched_barrier(0);
                    work(kb_c, m_c);
                    __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (kb == KA) second_loads();
                __builtin_amdgcn_sched_barrier(0);
            };
            block(I<0>{});
            if constexpr (NKB > 1) block(I<1>{});
            if constexpr (NKB > 2) block(I<2>{});
            if constexpr (NKB > 3) block(I<3>{});
            if constexpr (KB == NKB) { store_dy(v0, 2, buf ^ 1); store_x(v1, 0, hh_new, p.nnew); store_x(v2, 1, hh_new, p.nnew); }
            __syncthreads();
            buf ^= 1;
        }
    }

    // ---- sums that call for fp32 arithmetic: the work-group computes its share again (rule of split_finish) ----
    int col_j[3];                                                 // (c, r, s) of this lane's column, -1 where there is none
    int col_c[3], col_r[3], col_s[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const int quad = blk_col[b] * 8 + (l32 >> 2);
        const int cr = quad / p.SG, s = (quad - cr * p.SG) * 4 + (l32 & 3);
        const bool ok = quad < p.quads && s < p.S;
        col_j[b] = ok ? cr * p.S + s : -1;
        col_c[b] = ok ? cr / p.R : 0;
        col_r[b] = ok ? cr - cr / p.R * p.R : 0;
        col_s[b] = ok ? s : 0;
    }
    if (!stored4) col_j[2] = -1;
    auto tile_slot = [](int t) { return t < 3 ? t : t - 3; };
    auto tile_col = [](int t) { return t < 3 ? 0 : t - 2; };
    int *const words = reinterpret_cast<int *>(lds_fast);
    bool inf = false, nan = false;
#pragma unroll
    for (int t = 0; t < 5; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            acc[t][v] = (acc[t][v] + low[t][v]) * kSplitUnscale;
            const unsigned s = __float_as_uint(acc[t][v]);
            const bool here = col_j[tile_col(t)] >= 0 && slot_row[tile_slot(t)] * 32 + (v >> 2) * 8 + half * 4 + (v & 3) < p.K;
            inf |= here && (s & 0x7fffffffu) == 0x7f800000u;
            nan |= here && is_nan_bits(s);
        }
    const int f = split_group_or<NW>(words, wave, lane, (__ballot(inf) ? 1 : 0) | (__ballot(nan) ? 2 : 0));
    bool again = f & 1;
    // f(a, b) over this lane's operands: four pairs of positions at a time, this half's of each pair
    auto sweep = [&](auto use) {
#pragma unroll 1
        for (int unit = blockIdx.x; unit < p.units; unit += gridDim.x) {
            const int n = (int)fastdiv((uint32_t)unit, p.div_splits);
            const int sp = unit - n * p.splits;
            const int p_begin = (int)((int64_t)p.P * sp / p.splits), p_end = (int)((int64_t)p.P * (sp + 1) / p.splits);
#pragma unroll 1
            for (int prow = p_begin; prow < p_end; ++prow)
#pragma unroll 1
                for (int q0 = 0; q0 < p.Q; q0 += 8) {
                    float a[4][3], b[4][3];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const int q = q0 + 2 * t + half;
#pragma unroll
                        for (int i = 0; i < 3; ++i) {
                            const int m = slot_row[i] * 32 + l32;
                            const bool ok = q < p.Q && m < p.K;
                            a[t][i] = load_or_zero(p.dy, (int64_t)n * p.y_bs + ((int64_t)m * p.P + prow) * p.Q + q, ok);
                        }
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            const int h = 4 * prow + col_r[c] - p.pad, w = 4 * q + col_s[c] - p.pad;
                            const bool ok = q < p.Q && col_j[c] >= 0 && (unsigned)h < (unsigned)p.H && (unsigned)w < (unsigned)p.W;
                            b[t][c] = load_or_zero(p.x, (int64_t)n * p.x_bs + ((int64_t)col_c[c] * p.H + h) * p.W + w, ok);
                        }
                    }
                    if (!use(a, b)) return;
                }
        }
    };
    if (!again && (f & 2)) {
        int *const marks = words + 16;                            // rows with a NaN operand
        for (int i = tid; i < kRowsM; i += kRowsSplitThreads) marks[i] = 0;
        __syncthreads();
        int rows = 0, cols = 0;                                   // this lane's rows and columns with one, by slot
#pragma unroll
        for (int c = 0; c < 3; ++c) cols |= col_j[c] < 0 ? 1 << c : 0;
        sweep([&](const float (&a)[4][3], const float (&b)[4][3]) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    rows |= is_nan_bits(__float_as_uint(a[t][i])) ? 1 << i : 0;
                    cols |= is_nan_bits(__float_as_uint(b[t][i])) ? 1 << i : 0;
                }
            const int all_cols = cols | __shfl_xor(cols, 32);
            return !__all(all_cols == 7);                         // every column of the wave explains its sums
        });
        cols |= __shfl_xor(cols, 32);
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (rows >> i & 1) marks[slot_row[i] * 32 + l32] = 1;
        __syncthreads();
        bool open = false;
#pragma unroll
        for (int t = 0; t < 5; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = slot_row[tile_slot(t)] * 32 + (v >> 2) * 8 + half * 4 + (v & 3);
                open |= !(cols >> tile_col(t) & 1) && row < p.K && is_nan_bits(__float_as_uint(acc[t][v])) && !marks[row];
            }
        again = split_group_or<NW>(words, wave, lane, __ballot(open) ? 1 : 0) != 0;
    }
    if (again) {
#pragma unroll
        for (int t = 0; t < 5; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
        sweep([&](const float (&a)[4][3], const float (&b)[4][3]) {
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < 5; ++i)
                    acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t][tile_slot(i)], b[t][tile_col(i)], acc[i], 0, 0, 0);
            return true;
        });
    }

    float *const out = p.part + (size_t)blockIdx.x * p.K * p.Kg;
#pragma unroll
    for (int t = 0; t < 5; ++t) {
        const int j = col_j[tile_col(t)];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = slot_row[tile_slot(t)] * 32 + (v >> 2) * 8 + half * 4 + (v & 3);
            if (j >= 0 && row < p.K) out[(size_t)row * p.Kg + j] = acc[t][v];
        }
    }
}
