// fp32 backward-filter on the 16-bit matrix instructions, operands split into three bfloat16 parts (six products, two
// accumulators) or, where the tensors' range lets them, two half-precision parts (three products): see conv_split_kernels.h for
// the arithmetic, its error and its range.
// Part of convnet_hotpath.hip: included there, inside its anonymous namespace, after conv_split_kernels.h.
//
// dw[k][(r, s, c)] = sum over positions j = (n, p, q) of dy[n][k][p][q] * x[n][c][p*stride + r - pad][q*stride + s - pad].
// The matrix instruction wants eight consecutive positions of a row (filter or tap and channel) per lane, and NCHW tensors
// have them at odd addresses, so the tiles lie in LDS as [position][16 rows] and ds_read_b64_tr_b16 transposes them on
// the way into registers.  A staged piece is then 8 channels (filters) at ONE position: one padding test per piece, eight
// loads that are consecutive over the lanes of a wavefront, split in registers and written as 16 bytes per part.  There is
// no packed copy in memory (the workspace holds partial sums only, as for the fp32 kernels, whatever the mini-batch), and
// stride, padding and extents are free.
//
// One work-group (eight waves) per CU; a step covers 32 positions of a BM x BN tile: LDS block (16 rows of one part) =
// 32 positions x 32 bytes, two buffers of (BM + BN) * 192 bytes.  Position i of a block lies in slot i ^ 4 * (block & 1):
// the two blocks of a 32-row fragment are then read from different halves of the 64 banks.  In positions 4..7 of every eight
// the two 16-byte halves change places: eight lanes storing 16 bytes each then fall into different banks of 32.
// Order inside a step (two 16-position halves of six products each): the pieces of step + 1, loaded during the step before,
// are split and stored, and the loads of step + 2 issued, between the matrix instructions ahead of the barrier; the last
// two products of the step cover the barrier and the first fragment reads of the next.
//
// Measured (whole call): 384 -> 384 channels 3x3 on 13x13, N = 128: 625 -> 304 us; two columns 48 -> 128 5x5 on 27x27,
// N = 128: 640 -> 357 us (kernel 349: 267 TFLOP/s of six-product work at its padded 1280 columns); 384 -> 256, N = 33:
// 121 -> 77 us; error of that 384-channel layer's results against 64 bits 1.0e-6 -> 3.5e-7.  Bound: matrix instructions, 61 % of
// its cycles, no LDS bank conflicts; the six-product work and the splitting share the vector issue port.
// Two parts: half the matrix work, two thirds of the LDS traffic, 9 instead of 11 instructions to split a pair (the high halves
// by a packed conversion, the low ones by mixed-precision multiply-adds: with these for both, which issue at half rate, 215
// instead of 206 us).  The kernel of the 384-channel layer 310 -> 206 us.  Bound: no one unit but the sum of a wave's issue, 1100
// clocks of loads, splits, stores and reads beside 384 of matrix instructions each half step; of 215 us, without the loads 215,
// without splitting 190, without LDS reads 196, without stores 205, with one product of three 193.  One wave's matrix
// instructions against its neighbour's other work, a barrier a turn: 265.
//
// Loads are raw buffer loads: a piece outside the image or past the range of this split has its offset set past the
// descriptor's extent and reads as zero.

typedef short s16x4 __attribute__((ext_vector_type(4)));
struct WgradSplitArgs {
    const float *dy, *x;
    float *part;               // [nsplit][K][R*S*C], columns in (r, s, c) order
    int K, C, S, CB, ncols;    // CB: blocks of 16 channels; ncols = R*S*C
    int nblocks;               // R*S*CB: column blocks
    int P, Q, H, W, stride, pad;
    int dy_bs, x_bs;           // elements
    int J, steps_per_split;
    int mtiles, ntiles, nunits, units_per_xcd, nsplit;
    unsigned dy_bytes, x_bytes;       // bytes from a column's first element to its last
    int64_t dy_gs, x_gs, part_gs;     // elements between the columns of a grouped layer
    const SplitRanges *ranges;        // of dy and x, kernels with TWO
    float dense;
    FastDiv div_plane, div_q, div_cb, div_s;
};

// TAIL: K or C is no multiple of 16, so that a piece may reach past the end of its tensor: the channel's offset is then
// part of the checked offset instead of the scalar one.
// TWO: two half-precision parts where the operands' range lets it.
template <int TM, int TN, int WM, int WN, bool TWO> constexpr int wgrad_split_lds()
{
    const int rows = (TM * WM + TN * WN) * 32, three = 2 * rows * 192, two = 2 * rows * 128 + TM * TN * WM * WN * 64 * 32;
    return TWO && two > three ? two : three;
}
template <int TM, int TN, int WM, int WN, bool TAIL, bool TWO>
__global__ __launch_bounds__(WM * WN * 64, 1) void wgrad_split_kernel(const WgradSplitArgs p)
{
    constexpr int NW = WM * WN;
    constexpr int BM = TM * WM * 32, BN = TN * WN * 32;
    constexpr int QA = BM / 16, QB = BN / 16;                  // staged blocks per step
    constexpr int NT = (QA + QB + NW - 1) / NW;                // ... per wave
    constexpr int MPG = TM * TN;                               // matrix instructions per product
    static_assert(NW == 8, "eight waves");
    static_assert(wgrad_split_lds<TM, TN, WM, WN, TWO>() <= 160 * 1024, "LDS buffers");
    constexpr unsigned kOutside = 0x80000000u;

    extern __shared__ __attribute__((aligned(16))) float lds_fast[];
    char *const lds = reinterpret_cast<char *>(lds_fast);

    const int bid = blockIdx.x;
    const int idx = bid >> 3;
    const int unit = (bid & 7) * p.units_per_xcd + idx;
    if (idx >= p.units_per_xcd || unit >= p.nunits) return;
    const int tiles = p.mtiles * p.ntiles;
    const int gcol = unit / (tiles * p.nsplit);
    const int unit_c = unit - gcol * (tiles * p.nsplit);
    const int split = unit_c / tiles;
    const int tile = unit_c - split * tiles;
    const int mt = tile % p.mtiles, nt = tile / p.mtiles;
    const int m0 = mt * BM, n0 = nt * BN;

    const int tid = threadIdx.x, lane = tid & 63;
    SplitInfo info = {0, 0.f, 0.f, 0.f};
    if constexpr (TWO) info = split_info(p.ranges + gcol, lane, 2 * p.steps_per_split, p.dense);
    const int wave = uniform(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int PQ = p.P * p.Q;

    const int jbeg = split * p.steps_per_split * 32;
    const int jend = min(jbeg + p.steps_per_split * 32, p.J);
    const int nsteps = (jend - jbeg + 31) / 32;

    const float *const dyg = p.dy + (size_t)gcol * p.dy_gs;
    const float *const xg = p.x + (size_t)gcol * p.x_gs;

    f32x16 acc[TM][TN], low[TM][TN];           // sums of h h'; of the five smaller products
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int jn = 0; jn < TN; ++jn)
#pragma unroll
            for (int v = 0; v < 16; ++v) { acc[i][jn][v] = 0.f; low[i][jn][v] = 0.f; }

    const int l32 = lane & 31, half = lane >> 5;

    // column of this lane in block column jn of the wave: (r, s) tap and channel
    auto column = [&](int jn, int &rs, int &ch) {
        const int blk = n0 / 16 + (wn * TN + jn) * 2 + (l32 >> 4);
        rs = (int)fastdiv((uint32_t)blk, p.div_cb);
        ch = (blk - rs * p.CB) * 16 + (l32 & 15);
        return blk < p.nblocks && ch < p.C;
    };

    auto contract = [&](auto parts_c) {
    constexpr int PARTS = decltype(parts_c)::value;
    constexpr int BUF = (BM + BN) * PARTS * 64;

    const auto rsrc_dy = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(dyg), 0, (int)p.dy_bytes, 0x00020000);
    const auto rsrc_x = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(xg), 0, (int)p.x_bytes, 0x00020000);
    // of piece u: a wave's pieces are blocks of dy, then blocks of x; where the two meet inside a piece's row of waves, this wave's
    // choice is made here, once
    const auto rsrc_edge = [&](bool a) {   // by value: a conditional of the two names would keep both in memory
        if (a) return rsrc_dy;
        return rsrc_x;
    }(QA / NW * NW + wave < QA);
    auto rsrc_of = [&](int u) {
        if ((u + 1) * NW <= QA) return rsrc_dy;
        if (u * NW >= QA) return rsrc_x;
        return rsrc_edge;
    };

    // Piece u of this wave: block q = u * 8 + wave of the step (filters first), position lane % 32, rows
    // (lane / 32) * 8 .. + 7 of the block.
    const int pos = lane & 31, oct = lane >> 5;
    bool isa[NT], none[NT];
    int tap_r[NT], tap_s[NT];
    unsigned row_off[NT], st_off[NT];                          // bytes: first row's plane; LDS address of part 0
#pragma unroll
    for (int u = 0; u < NT; ++u) {
        const int q = u * NW + wave;
        isa[u] = (u + 1) * NW <= QA || (u * NW < QA && q < QA);
        none[u] = (u + 1) * NW > QA + QB && q >= QA + QB;
        tap_r[u] = tap_s[u] = 0;
        if (isa[u]) {
            const int k0 = min(m0 / 16 + q, (p.K + 15) / 16 - 1) * 16;       // blocks past the last: computed, never stored
            row_off[u] = (unsigned)(k0 + oct * 8) * (unsigned)(PQ * 4);
            st_off[u] = (unsigned)(q * 1024 + (pos ^ ((q & 1) * 4)) * 32 + (oct ^ ((pos >> 2) & 1)) * 16);
        } else {
            const int b = none[u] ? 0 : q - QA;
            const int blk = min(n0 / 16 + b, p.nblocks - 1);
            const int rs = (int)fastdiv((uint32_t)blk, p.div_cb), cb = blk - rs * p.CB;
            tap_r[u] = (int)fastdiv((uint32_t)rs, p.div_s);
            tap_s[u] = rs - tap_r[u] * p.S;
            row_off[u] = (unsigned)(cb * 16 + oct * 8) * (unsigned)(p.H * p.W * 4);
            st_off[u] = (unsigned)(BM * (PARTS * 64) + b * 1024 + (pos ^ ((b & 1) * 4)) * 32 + (oct ^ ((pos >> 2) & 1)) * 16);
        }
    }

    float st[NT][8];
    int jnext = jbeg + pos;
    // where this lane's position of the next step to load sits
    unsigned ybase = 0, xbase = 0;
    int hb = 0, wb = 0;
    auto next_position = [&]() {
        const bool ok = jnext < jend;
        const int js = ok ? jnext : jbeg;
        const int n = (int)fastdiv((uint32_t)js, p.div_plane);
        const int pq = js - n * PQ;
        const int pp = (int)fastdiv((uint32_t)pq, p.div_q);
        hb = pp * p.stride - p.pad;
        wb = (pq - pp * p.Q) * p.stride - p.pad;
        ybase = ok ? (unsigned)(n * p.dy_bs + pq) * 4u : kOutside;
        xbase = (unsigned)(n * p.x_bs + hb * p.W + wb) * 4u;       // may wrap below zero: only used inside the image
        if (!ok) hb = kInvalidTap;
        jnext += 32;
    };
    unsigned voff[NT];
    auto piece_offset = [&](int u) {
        if (isa[u]) {
            voff[u] = ybase == kOutside ? kOutside : ybase + row_off[u];
        } else {
            const bool in = (unsigned)(hb + tap_r[u]) < (unsigned)p.H && (unsigned)(wb + tap_s[u]) < (unsigned)p.W;
            voff[u] = in ? xbase + (unsigned)(tap_r[u] * p.W + tap_s[u]) * 4u + row_off[u] : kOutside;
        }
    };
    auto load_one = [&](int u, int k) {
        if (none[u]) return;
        const int plane = (isa[u] ? PQ : p.H * p.W) * 4;
        const auto rsrc = rsrc_of(u);
        // outside: 0x80000000 + 7 * plane stays past the extent (tensors and planes are shorter than 2^31 bytes together)
        const unsigned v = TAIL ? voff[u] + (unsigned)(k * plane) : voff[u];
        st[u][k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, v, TAIL ? 0 : k * plane, 0));
    };
    u32x4 sp[PARTS];
    auto split_two = [&](int u, int t) {
        if (none[u]) return;
        unsigned h, m, l;
        if constexpr (PARTS == 2) {
            const float s = isa[u] ? info.sa : info.sb;
            split_pair_two(st[u][2 * t], st[u][2 * t + 1], s, s * kHalfLow, h, l);
            sp[0][t] = h; sp[1][t] = l;
        } else {
            split_pair(st[u][2 * t], st[u][2 * t + 1], h, m, l);
            sp[0][t] = h; sp[1][t] = m; sp[2][t] = l;
        }
    };
    auto store_piece = [&](int u, int buf) {
        if (none[u]) return;
        const int part_bytes = (isa[u] ? QA : QB) * 1024;
        char *const d = lds + buf * BUF + st_off[u];
#pragma unroll
        for (int c = 0; c < PARTS; ++c) *reinterpret_cast<u32x4 *>(d + c * part_bytes) = sp[c];
    };
    auto load_step = [&]() {
        next_position();
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            piece_offset(u);
#pragma unroll
            for (int k = 0; k < 8; ++k) load_one(u, k);
        }
    };

    // Fragment reads: the 16 lanes of group g = lane / 16 read four positions of block g % 2; lanes 0..31 hold positions
    // 0..7 of a half step, lanes 32..63 positions 12..15 and 8..11 (the same order for both operands).
    const int sub = (lane >> 4) & 1;
    const unsigned frag0 = (unsigned)(sub * 1024 + ((((half ? 12 : 0)) ^ (sub * 4)) + ((lane & 15) >> 2)) * 32 +
                                      ((lane & 3) ^ (half * 2)) * 8);
    typedef __attribute__((address_space(3))) char *lds_bytes;
    typedef __attribute__((address_space(3))) s16x4 *lds_quad;
    const lds_bytes frag_lo = (lds_bytes)lds + frag0, frag_hi = (lds_bytes)lds + (frag0 ^ 144u);   // 4 positions on
    const int a_frag = wm * TM * 2 * 1024, b_frag = BM * (PARTS * 64) + wn * TN * 2 * 1024;
    auto read_tr = [&](int off) {
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad)(frag_lo + off));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad)(frag_hi + off));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    typedef decltype(__builtin_shufflevector(s16x4{}, s16x4{}, 0, 1, 2, 3, 4, 5, 6, 7)) frag_t;
    load_step();
#pragma unroll
    for (int u = 0; u < NT; ++u) {
#pragma unroll
        for (int t = 0; t < 4; ++t) split_two(u, t);
        store_piece(u, 0);
    }
    load_step();
    next_position();
    __syncthreads();
    if constexpr (PARTS == 2) {
        // A half step: h h' and h l', the barrier at the end of a step, the next half's h and h' into the other set, l h'
        frag_t ha[2][TM], hb[2][TN], la[TM], lb[TN];
        auto read = [&](int buf, int t, int c, frag_t (&a)[TM], frag_t (&b)[TN]) {
#pragma unroll
            for (int i = 0; i < TM; ++i) a[i] = read_tr(a_frag + buf * BUF + t * 512 + (c * QA + i * 2) * 1024);
#pragma unroll
            for (int jn = 0; jn < TN; ++jn) b[jn] = read_tr(b_frag + buf * BUF + t * 512 + (c * QB + jn * 2) * 1024);
        };
        read(0, 0, 0, ha[0], hb[0]);
        char *const aside = lds + 2 * BUF + tid * 16;
        split_clear_aside<NW, TM, TN>(aside);
        const int segment = nsteps / info.segments;
        int segment_end = segment;
        constexpr int SLOTS = 5 * MPG, WORK = NT * 13, PER = (WORK + SLOTS - 1) / SLOTS;
        for (int step = 0; step < nsteps; ++step) {
            const int buf = step & 1;
            if (step >= segment_end) {
                split_put_aside<NW>(acc, aside);
                segment_end += segment;
            }
            auto work = [&](auto i_c) {
                // a piece's thirteen: S0 L0 L1 S1 L2 L3 S2 L4 L5 S3 store L6 L7 (a load goes where its registers have been split)
                constexpr int u = decltype(i_c)::value / 13, s = decltype(i_c)::value % 13;
                if constexpr (u < NT) {
                    if constexpr (s == 0) piece_offset(u);
                    if constexpr (s % 3 == 0 && s < 12) split_two(u, s / 3);
                    else if constexpr (s == 10) store_piece(u, buf ^ 1);
                    else load_one(u, s < 10 ? s / 3 * 2 + s % 3 - 1 : s - 5);
                }
            };
            auto product = [&](const frag_t (&xa)[TM], const frag_t (&xb)[TN], auto g_c) {
                constexpr int g = decltype(g_c)::value;
                static_for<MPG>([&](auto q_c) {
                    constexpr int i = decltype(q_c)::value / TN, jn = decltype(q_c)::value % TN, m = g * MPG + decltype(q_c)::value;
                    f32x16 &sum = g % 3 == 0 ? acc[i][jn] : low[i][jn];
                    sum = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, xa[i]), __builtin_bit_cast(f16x8, xb[jn]),
                                                                 sum, 0, 0, 0);
                    if constexpr (m < SLOTS && m * PER < WORK) {
                        __builtin_amdgcn_sched_barrier(0);
                        static_for<PER>([&](auto w_c) { work(I<m * PER + decltype(w_c)::value>{}); });
                        __builtin_amdgcn_sched_barrier(0);
                    }
                });
                __builtin_amdgcn_sched_barrier(0);
            };
            auto half_step = [&](auto t_c) {
                constexpr int t = decltype(t_c)::value;
                read(buf, t, 1, la, lb);
                __builtin_amdgcn_sched_barrier(0);
                product(ha[t], hb[t], I<t * 3>{});
                product(ha[t], lb, I<t * 3 + 1>{});
                if constexpr (t == 1) {
                    asm volatile("s_waitcnt lgkmcnt(0)");
                    __syncthreads();
                    __builtin_amdgcn_sched_barrier(0);
                }
                read(t == 1 ? buf ^ 1 : buf, t ^ 1, 0, ha[t ^ 1], hb[t ^ 1]);
                __builtin_amdgcn_sched_barrier(0);
                product(la, hb[t], I<t * 3 + 2>{});
                if constexpr (t == 1) next_position();
            };
            half_step(I<0>{});
            half_step(I<1>{});
        }
        split_take_back<NW>(acc, low, aside, info.unscale);
    } else {
    frag_t fa[3][TM], fb[3][TN];
    auto read_a = [&](int buf, int t, int c) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[c][i] = read_tr(a_frag + buf * BUF + t * 512 + (c * QA + i * 2) * 1024);
    };
    auto read_b = [&](int buf, int t, int c) {
#pragma unroll
        for (int jn = 0; jn < TN; ++jn) fb[c][jn] = read_tr(b_frag + buf * BUF + t * 512 + (c * QB + jn * 2) * 1024);
    };

    read_a(0, 0, 0);
    read_b(0, 0, 0);

    // Work between the matrix instructions ahead of the barrier: per piece four splits, its store and eight loads
    constexpr int SLOTS = 10 * MPG;                            // matrix instructions before the barrier
    constexpr int WORK = NT * 13;
    constexpr int PER = (WORK + SLOTS - 1) / SLOTS;
    for (int step = 0; step < nsteps; ++step) {
        const int buf = step & 1;
        auto work = [&](auto i_c) {
            // a piece's thirteen: S0 L0 L1 S1 L2 L3 S2 L4 L5 S3 store L6 L7 (a load goes where its registers have been split)
            constexpr int u = decltype(i_c)::value / 13, s = decltype(i_c)::value % 13;
            if constexpr (u < NT) {
                if constexpr (s == 0) piece_offset(u);
                if constexpr (s % 3 == 0 && s < 12) split_two(u, s / 3);
                else if constexpr (s == 10) store_piece(u, buf ^ 1);
                else load_one(u, s < 10 ? s / 3 * 2 + s % 3 - 1 : s - 5);
            }
        };
        auto product = [&](auto ca_c, auto cb_c, auto g_c) {   // parts of the filters' and the inputs' side; product 0..11
            constexpr int ca = decltype(ca_c)::value, cb = decltype(cb_c)::value, g = decltype(g_c)::value;
            static_for<MPG>([&](auto q_c) {
                constexpr int i = decltype(q_c)::value / TN, jn = decltype(q_c)::value % TN, m = g * MPG + decltype(q_c)::value;
                f32x16 &sum = g % 6 == 0 ? acc[i][jn] : low[i][jn];
                sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa[ca][i]),
                                                              __builtin_bit_cast(bf16x8, fb[cb][jn]), sum, 0, 0, 0);
                if constexpr (m < SLOTS && m * PER < WORK) {
                    __builtin_amdgcn_sched_barrier(0);
                    static_for<PER>([&](auto w_c) { work(I<m * PER + decltype(w_c)::value>{}); });
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
            __builtin_amdgcn_sched_barrier(0);
        };
        auto half_step = [&](auto t_c) {
            constexpr int t = decltype(t_c)::value, next_t = t ^ 1;
            const int next_buf = t == 1 ? buf ^ 1 : buf;
            read_b(buf, t, 2);
            read_a(buf, t, 2);
            __builtin_amdgcn_sched_barrier(0);
            product(I<0>{}, I<0>{}, I<t * 6>{});
            read_b(buf, t, 1);
            read_a(buf, t, 1);
            __builtin_amdgcn_sched_barrier(0);
            product(I<0>{}, I<2>{}, I<t * 6 + 1>{});
            product(I<2>{}, I<0>{}, I<t * 6 + 2>{});
            product(I<0>{}, I<1>{}, I<t * 6 + 3>{});
            if (t == 1) {
                asm volatile("s_waitcnt lgkmcnt(0)");
                __syncthreads();
                __builtin_amdgcn_sched_barrier(0);
            }
            read_a(next_buf, next_t, 0);
            __builtin_amdgcn_sched_barrier(0);
            product(I<1>{}, I<0>{}, I<t * 6 + 4>{});
            if (t == 1) next_position();
            read_b(next_buf, next_t, 0);
            __builtin_amdgcn_sched_barrier(0);
            product(I<1>{}, I<1>{}, I<t * 6 + 5>{});
        };
        half_step(I<0>{});
        half_step(I<1>{});
    }

    // sums that call for fp32 arithmetic: the whole work-group computes its tile again
    {
        bool col_ok[TN];
#pragma unroll
        for (int jn = 0; jn < TN; ++jn) {
            int rs, ch;
            col_ok[jn] = column(jn, rs, ch);
        }
        auto scan = [&](int *nan_rows, int *nan_cols) {
            jnext = jbeg + pos;
            for (int step = 0; step < nsteps; ++step) {
                next_position();
#pragma unroll
                for (int u = 0; u < NT; ++u) {
                    if (none[u]) continue;
                    const int plane = (isa[u] ? PQ : p.H * p.W) * 4, b = u * NW + wave;
                    const auto rsrc = rsrc_of(u);
                    int *const mark = (isa[u] ? nan_rows + b * 16 : nan_cols + (b - QA) * 16) + oct * 8;
                    piece_offset(u);
                    unsigned nans = 0;
#pragma unroll
                    for (int k = 0; k < 8; ++k)
                        nans |= is_nan_bits(__builtin_amdgcn_raw_buffer_load_b32(rsrc, TAIL ? voff[u] + (unsigned)(k * plane) : voff[u],
                                                                                 TAIL ? 0 : k * plane, 0)) ? 1u << k : 0u;
                    for (int k = 0; k < 8; ++k)
                        if (nans >> k & 1) mark[k] = 1;
                }
            }
        };
        if (split_finish<TM, TN, NW, BM, BN>(acc, low, wm * TM * 32 + half * 4, p.K - m0, wn * TN * 32 + l32, col_ok,
                                             reinterpret_cast<int *>(lds_fast), wave, lane, scan)) {
            int tr[TN], ts[TN];
            int64_t boff[TN];
            bool bok[TN];
#pragma unroll
            for (int jn = 0; jn < TN; ++jn) {
                int rs, ch;
                bok[jn] = column(jn, rs, ch);
                tr[jn] = (int)fastdiv((uint32_t)rs, p.div_s);
                ts[jn] = rs - tr[jn] * p.S;
                boff[jn] = (int64_t)ch * (p.H * p.W);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int jn = 0; jn < TN; ++jn)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][jn][v] = 0.f;
#pragma unroll 1
            for (int j0 = jbeg; j0 < jend; j0 += 8) {            // the loads of eight positions in flight, unconditional
                float a[4][TM], b[4][TN];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int j = j0 + t * 2 + half;
                    const bool jok = j < jend;
                    const int js = jok ? j : jbeg;
                    const int n = (int)fastdiv((uint32_t)js, p.div_plane);
                    const int pq = js - n * PQ;
                    const int pp = (int)fastdiv((uint32_t)pq, p.div_q);
                    const int h0 = pp * p.stride - p.pad, w0 = (pq - pp * p.Q) * p.stride - p.pad;
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        const int k = m0 + (wm * TM + i) * 32 + l32;
                        const float e = dyg[(int64_t)n * p.dy_bs + (int64_t)min(k, p.K - 1) * PQ + pq];
                        a[t][i] = jok && k < p.K ? e : 0.f;
                    }
#pragma unroll
                    for (int jn = 0; jn < TN; ++jn) {
                        const int h = h0 + tr[jn], w = w0 + ts[jn];
                        const bool ok = jok && bok[jn] && (unsigned)h < (unsigned)p.H && (unsigned)w < (unsigned)p.W;
                        const float e = xg[ok ? (int64_t)n * p.x_bs + boff[jn] + h * p.W + w : 0];
                        b[t][jn] = ok ? e : 0.f;
                    }
                }
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int i = 0; i < TM; ++i)
#pragma unroll
                        for (int jn = 0; jn < TN; ++jn)
                            acc[i][jn] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t][i], b[t][jn], acc[i][jn], 0, 0, 0);
            }
        }
    }

    }
    };
    if constexpr (TWO) {
        if (info.segments) contract(I<2>{});
        else contract(I<3>{});
    } else {
        contract(I<3>{});
    }

    float *const out = p.part + (size_t)gcol * p.part_gs + (size_t)split * p.K * p.ncols;
#pragma unroll
    for (int jn = 0; jn < TN; ++jn) {
        int rs, ch;
        if (!column(jn, rs, ch)) continue;
        const int col = rs * p.C + ch;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int row0 = m0 + (wm * TM + i) * 32 + half * 4;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = row0 + (v >> 2) * 8 + (v & 3);
                if (row < p.K) out[(size_t)row * p.ncols + col] = acc[i][jn][v];
            }
        }
    }
}
