// Stride-1 forward / backward-data with bf16 inputs for layers of few channels or few GEMM rows (the second layer's columns:
// 48 -> 128 channels 5x5): the input window of a tile stays in LDS while all filter taps pass over it.
// Part of convnet_hotpath.hip: included there, inside its anonymous namespace, after conv_bf16_dma_kernels.h.
//
// Why: a kernel that loads its activations per tap brings every input element R*S times through the vector memory path (and
// the register-staged one also through LDS stores), which at 48 GEMM rows or 48 channels is far more time than the matrix
// work.  Here the padded rows under a tile of output positions come in once per channel block, by linear direct-to-LDS loads,
// and a tap is an address offset of the fragment reads.
//
// Layouts that window_prepare writes:
//   xb  [channel block of 16][n][Hp][Wp][16 channels]: the padded rows of consecutive samples follow each other, so the rows
//       under consecutive output positions (n, oh, ow) are one run of memory.  The two 16-byte halves of a position change
//       places where bit 3 of its number (n Hp + hp) Wp + wp is set: 16 lanes that read 16 consecutive positions, from
//       whichever one on, then cover the 64 banks.  Runs start at a multiple of 16 positions, so the same bit of the position
//       in the window says so.
//   wt  [channel chunk][tap, in the order of window offsets][block of the chunk][Mpad][16 channels], halves swapped by bit 3 of
//       the row: linear in memory and in LDS.
// The columns of a grouped layer follow each other in both; channel blocks are padded with zeros to whole chunks of NCB.
//
// A step is one tap (MULTI: two) x NCB channel blocks.  Layers of one chunk hold one window and two filter buffers, so that two
// work-groups of four waves share a CU and hide each other's window loads.  Others (MULTI) prefetch the next chunk's window
// into a second buffer and keep the filters of two steps in flight in three buffers; that fills the LDS, so the work-group has
// eight waves, two per SIMD: waves 0..3 take the even taps, waves 4..7 the odd ones, and the two sums of a tile are added
// through LDS at the end, each group finishing half of the rows.  (With four waves the loop took 91k clocks where the matrix
// work is 38k: one wave per SIMD waits for each of its LDS reads.)
// A wave owns 64 rows x 32 TN positions: with TN = 3 it reads five fragments for six matrix instructions.
// Two columns 48 -> 128 channels 5x5 on 27x27, both together, preparation + kernel, against the register-staged kernel: forward
// N = 64 57 -> 41 us (9 + 32), N = 128 94 -> 70; backward-data N = 64 79 -> 54 (12 + 42), N = 128 137 -> 98.  Bound: matrix
// instructions in the loop; of the cycles in which a CU holds work-groups the matrix unit is busy 56 % forward and 49 % backward-data
// (N = 64), the others being set-up, first window and stores.  Backward-data pads 48 rows to 64.  10 % of the cycles are LDS
// bank conflicts.  The preparation is bound by memory (5 TB/s at N = 128).

struct ColGemmWindowArgs {
    const char *At, *xb;
    void *dst;                               // y or dx: fp32, or bfloat16 when out_bf16
    int M, Mpad, ncols;
    int OH, OW, Hp, Wp, R, S;
    int chunks;                              // channel chunks per column
    unsigned cb_bytes;                       // one channel block: N * Hp * Wp * 32
    int win_bytes;                           // LDS bytes of one block's window, a multiple of 1024
    int mtiles, ntiles, tiles_per_xcd, groups;
    int64_t at_gb, dst_gs;                   // bytes of a column's filters; elements between its outputs
    int dst_bs, out_bf16;
    int epi_on;
    Epilogue epi;
    FastDiv div_plane, div_ow;
};

template <int TN, int WM, int WN, int NCB, bool MULTI>
__global__ __launch_bounds__(MULTI ? 512 : 256, MULTI ? 1 : 2) void colgemm_bf16_window_kernel(const ColGemmWindowArgs p)
{
    constexpr int TM = 2, KG = MULTI ? 2 : 1, NW = 4 * KG;       // KG: groups of four waves that share out the taps
    constexpr int BM = TM * WM * 32, BN = TN * WN * 32;
    constexpr int NBUF = MULTI ? 3 : 2;
    constexpr int AQ = NCB * BM / 32;                            // 1 KB blocks of filters per tap
    constexpr int NLA = (AQ + 3) / 4;                            // ... per wave and step (the last may repeat an earlier one)
    constexpr int ABUF = KG * AQ * 1024;
    constexpr int NLW = NCB;                                     // loads of the next window per wave and step
    static_assert(WM * WN == 4, "four waves");

    extern __shared__ __attribute__((aligned(16))) float lds_fast[];
    char *const lds = reinterpret_cast<char *>(lds_fast);        // filter buffers | window buffers
    const unsigned lds_base = (unsigned)(size_t)lds_fast;

    const int bid = blockIdx.x;
    const int idx = bid >> 3;
    const int unit = (bid & 7) * p.tiles_per_xcd + idx;
    const int ntile = p.mtiles * p.ntiles;
    if (idx >= p.tiles_per_xcd || unit >= ntile * p.groups) return;
    const int gcol = unit / ntile;
    const int tile = unit - gcol * ntile;
    const int mt = tile % p.mtiles, nt = tile / p.mtiles;
    const int m0 = mt * BM, n0 = nt * BN;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = uniform(tid >> 6), kg = MULTI ? wave >> 2 : 0, w4 = wave & 3;
    const int wm = w4 / WN, wn = w4 % WN;
    const int l32 = lane & 31, half = lane >> 5;

    // number of output position j's window origin among the padded positions
    auto origin = [&](int j) {
        const int n = (int)fastdiv((uint32_t)j, p.div_plane);
        const int rem = j - n * (p.OH * p.OW);
        const int oh = (int)fastdiv((uint32_t)rem, p.div_ow);
        return (n * p.Hp + oh) * p.Wp + (rem - oh * p.OW);
    };
    const int start = origin(n0) & ~15;
    const int end = origin(min(n0 + BN, p.ncols) - 1) + (p.R - 1) * p.Wp + p.S;        // one past the last position read
    // 1 KB loads of a block's window, in rounds of one per wave (with MULTI a round may reach past the window, into what
    // follows it, so that every wave has the same number of loads in flight)
    const int kilobytes = uniform(((end - start) * 32 + 1023) / 1024), rounds = (kilobytes + NW - 1) / NW;
    const char *const xb = p.xb + (size_t)gcol * p.chunks * NCB * p.cb_bytes + (size_t)start * 32;
    const int taps = p.R * p.S, chunk_steps = (taps + KG - 1) / KG, steps = p.chunks * chunk_steps;
    const unsigned w_voff = (unsigned)(wave * 1024 + lane * 16);
    const unsigned w_lds = lds_base + NBUF * ABUF + wave * 1024;
    // filters: each group loads its tap's, 1 KB blocks of 32 rows
    unsigned a_voff[NLA], a_lds[NLA];
#pragma unroll
    for (int i = 0; i < NLA; ++i) {
        int q = i * 4 + w4;
        if (q >= AQ) q -= 4;
        const int b = q / (BM / 32), r = q - b * (BM / 32);
        a_voff[i] = (unsigned)((kg * NCB + b) * p.Mpad * 32 + r * 1024 + lane * 16);
        a_lds[i] = lds_base + (kg * AQ + q) * 1024;
    }
    const size_t a_step = (size_t)KG * NCB * p.Mpad * 32, a_last = a_step - (size_t)(chunk_steps * KG - taps) * NCB * p.Mpad * 32;
    const char *a_next = p.At + (size_t)gcol * p.at_gb + (size_t)m0 * 32;              // filters of the next step to load
    int a_left = chunk_steps;
    auto load_a = [&](int i, unsigned buf) { dma16(a_next, a_voff[i], a_lds[i] + buf); };
    auto advance_a = [&]() {
        if (KG > 1 && --a_left == 0) { a_left = chunk_steps; a_next += a_last; }
        else a_next += a_step;
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int jn = 0; jn < TN; ++jn)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][jn][v] = 0.f;

    const int a_row = kg * AQ * 1024 + (wm * TM * 32 + l32) * 32 + (half ^ ((l32 >> 3) & 1)) * 16;
    unsigned pos[TN];                                            // byte offset of this lane's position, half in bit 4
#pragma unroll
    for (int jn = 0; jn < TN; ++jn)
        pos[jn] = (unsigned)(origin(min(n0 + (wn * TN + jn) * 32 + l32, p.ncols - 1)) - start) * 32u + half * 16u;

    u32x4 fa[2][TM], fb[2][TN];
    unsigned badr[TN], aadr;                                     // LDS offsets under the current tap, block 0
    auto set_tap = [&](unsigned tap_off, unsigned abuf) {        // tap_off: bytes, window buffer and filter buffers included
        aadr = a_row + abuf;
#pragma unroll
        for (int jn = 0; jn < TN; ++jn) {
            const unsigned a = pos[jn] + tap_off;
            badr[jn] = a ^ ((a >> 4) & 16u);
        }
    };
    auto read_frags = [&](int b, int set) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[set][i] = *reinterpret_cast<const u32x4 *>(lds + aadr + (b * BM + i * 32) * 32);
#pragma unroll
        for (int jn = 0; jn < TN; ++jn) fb[set][jn] = *reinterpret_cast<const u32x4 *>(lds + badr[jn] + b * p.win_bytes);
    };

    for (int b = 0; b < NCB; ++b)
        for (int i = 0; i < rounds; ++i)
            if (MULTI || i * NW + wave < kilobytes)
                dma16(xb + (size_t)b * p.cb_bytes + (size_t)i * (NW * 1024), w_voff, w_lds + b * p.win_bytes + i * (NW * 1024));
#pragma unroll
    for (int t = 0; t < NBUF - 1; ++t) {
#pragma unroll
        for (int i = 0; i < NLA; ++i) load_a(i, t * ABUF);
        advance_a();
    }
    wait_vmcnt<0>();
    __syncthreads();

    // One step: NCB slices; the fragments of the next slice are read while one is multiplied, and the loads go out between
    // the first slice's matrix instructions.  Before the last slice: wait for the filters of step + 1 (issued a step
    // earlier with three buffers, in this step with two) and, a chunk's last two steps carrying none, for the whole next
    // window; barrier; first reads of the next step.  Filters past the last step are loaded (there is room behind them in the
    // workspace) and not used, so that the number of loads in flight is known; so are the reads of the step after the last.
    // A wave has little else to issue beside its matrix instructions: offsets move on by additions.
    constexpr unsigned kFirstWindow = NBUF * ABUF;
    const unsigned win_buf = (unsigned)(NCB * p.win_bytes);
    unsigned tap_off = kFirstWindow + kg * 32u, abuf = 0, aload = (NBUF - 1) * ABUF;
    int step = 0, s_left = p.S - kg, chunk_left = chunk_steps, tap = kg;
    // next chunk's window: loads left, of the block that is being loaded, where from and where to
    int w_left = MULTI && p.chunks > 1 ? NCB * rounds : 0, w_block = rounds, chunk = 0;
    const char *w_src = xb + (size_t)NCB * p.cb_bytes;
    unsigned w_dst = w_lds + win_buf, wbuf = 0;
    const size_t w_hop = p.cb_bytes - (size_t)(rounds - 1) * (NW * 1024);
    const unsigned w_hop_lds = (unsigned)(p.win_bytes - (rounds - 1) * (NW * 1024));
    set_tap(tap_off, 0);
    read_frags(0, 0);
    auto do_step = [&](auto par_c) {
        constexpr int par = decltype(par_c)::value;
        const bool more_w = MULTI && w_left > 0;
        const bool real = KG == 1 || tap < taps;                 // an odd count of taps: the second group's last is none (the
                                                                 // LDS goes on a row behind the last window for its reads)
#pragma unroll
        for (int b = 0; b < NCB; ++b) {
            const int set = (par + b) & 1;
            if (b + 1 < NCB) {
                read_frags(b + 1, set ^ 1);
            } else {
                if (!MULTI) wait_vmcnt<0>();
                else if (more_w) wait_vmcnt<NLA + NLW>();
                else wait_vmcnt<NLA>();
                asm volatile("s_waitcnt lgkmcnt(0)");
                __syncthreads();
                tap_off += KG * 32;
                tap += KG;
                if ((s_left -= KG) <= 0) { s_left += p.S; tap_off += (unsigned)(p.Wp - p.S) * 32u; }
                if (MULTI && --chunk_left == 0) {
                    chunk_left = chunk_steps;
                    wbuf = win_buf - wbuf;
                    tap_off = kFirstWindow + wbuf + kg * 32u;
                    s_left = p.S - kg;
                    tap = kg;
                    ++chunk;
                    w_left = chunk + 1 < p.chunks ? NCB * rounds : 0;
                    w_block = rounds;
                    w_src = xb + (size_t)(chunk + 1) * NCB * p.cb_bytes;
                    w_dst = w_lds + win_buf - wbuf;
                }
                abuf = abuf == (NBUF - 1) * ABUF ? 0 : abuf + ABUF;
                set_tap(tap_off, abuf);
                read_frags(0, set ^ 1);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (b == 0) {
#pragma unroll
                for (int i = 0; i < NLA; ++i) load_a(i, aload);
                if (MULTI && more_w) {
#pragma unroll
                    for (int i = 0; i < NLW; ++i) {              // (NCB * rounds is a multiple of NLW)
                        dma16(w_src, w_voff, w_dst);
                        --w_left;
                        if (--w_block == 0) { w_block = rounds; w_src += w_hop; w_dst += w_hop_lds; }
                        else { w_src += NW * 1024; w_dst += NW * 1024; }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (real)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int jn = 0; jn < TN; ++jn)
                        acc[i][jn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa[set][i]),
                                                                             __builtin_bit_cast(bf16x8, fb[set][jn]),
                                                                             acc[i][jn], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        advance_a();
        aload = aload == (NBUF - 1) * ABUF ? 0 : aload + ABUF;
        ++step;
    };
    if (NCB % 2 == 0) {
        while (step < steps) do_step(std::integral_constant<int, 0>{});
    } else {
        while (step + 1 < steps) {
            do_step(std::integral_constant<int, 0>{});
            do_step(std::integral_constant<int, 1>{});
        }
        if (step < steps) do_step(std::integral_constant<int, 0>{});
    }
    wait_vmcnt<0>();

    constexpr int TF = TM / KG;                                  // blocks of 32 rows that a wave finishes
    f32x16 fin[TF][TN];
    if constexpr (KG == 1) {
#pragma unroll
        for (int i = 0; i < TF; ++i)
#pragma unroll
            for (int jn = 0; jn < TN; ++jn) fin[i][jn] = acc[i][jn];
    } else {
        // each group hands over the sums of the rows that the other finishes
        f32x4 *const trade = reinterpret_cast<f32x4 *>(lds) + (size_t)w4 * (TN * 4 * 64) + lane;
        constexpr int side = 4 * TN * 4 * 64;
        __syncthreads();
#pragma unroll
        for (int jn = 0; jn < TN; ++jn) {
            const f32x16 a = acc[0][jn], b = acc[1][jn];         // (by value: a choice of arrays would keep both in memory)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                f32x4 other;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    other[e] = kg == 0 ? b[4 * v + e] : a[4 * v + e];
                    fin[0][jn][4 * v + e] = kg == 0 ? a[4 * v + e] : b[4 * v + e];
                }
                trade[(kg ^ 1) * side + (jn * 4 + v) * 64] = other;
            }
        }
        __syncthreads();
#pragma unroll
        for (int jn = 0; jn < TN; ++jn)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const f32x4 o = trade[kg * side + (jn * 4 + v) * 64];
#pragma unroll
                for (int e = 0; e < 4; ++e) fin[0][jn][4 * v + e] += o[e];
            }
    }

    // Stores: offsets from the tensor's first byte fit 32 bits (checked spans).
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const int plane = p.OH * p.OW, row0 = m0 + wm * TM * 32 + kg * 32 + half * 4;
#pragma unroll
    for (int jn = 0; jn < TN; ++jn) {
        const int col = n0 + (wn * TN + jn) * 32 + l32;
        const bool in = col < p.ncols;
        const int n = (int)fastdiv((uint32_t)(in ? col : p.ncols - 1), p.div_plane);
        const int rem = (in ? col : p.ncols - 1) - n * plane;
        if (p.epi_on) epi_tile<TF, TN>(p.epi, fin, jn, row0, p.M, plane, (int64_t)n * p.epi.mask_bs + rem);
        const unsigned own = (unsigned)n * (unsigned)p.dst_bs + (unsigned)rem + (unsigned)row0 * (unsigned)plane;
        int left = in ? p.M - row0 : 0;
        asm volatile("" : "+v"(left));           // or the rows' masks are kept in registers over the columns
        if (!p.out_bf16) {
            char *const out = reinterpret_cast<char *>(static_cast<float *>(p.dst) + (size_t)gcol * p.dst_gs);
#pragma unroll
            for (int i = 0; i < TF; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int d = i * 32 + (v >> 2) * 8 + (v & 3);
                    if (d < left) *reinterpret_cast<float *>(out + (4u * (own + (unsigned)(d * plane)))) = fin[i][jn][v];
                }
            continue;
        }
        // Neighbouring lanes (positions col, col + 1 of one sample) trade a value so that the even lane stores row a of both
        // positions and the odd lane row a + 1 of both, four bytes each; lanes whose neighbour belongs to another sample, or
        // lies past the last column, store their two values one by one.
        char *const out = reinterpret_cast<char *>(static_cast<unsigned short *>(p.dst) + (size_t)gcol * p.dst_gs);
        const bool odd = l32 & 1;
        const bool pair = odd ? rem >= 1 : rem + 1 < plane && col + 1 < p.ncols;
        const unsigned both = own + (odd ? (unsigned)plane - 1u : 0u);
        const int left_both = left - (odd ? 1 : 0);
#pragma unroll
        for (int i = 0; i < TF; ++i)
#pragma unroll
            for (int v = 0; v < 16; v += 2) {
                const int d = i * 32 + (v >> 2) * 8 + (v & 3);
                const float va = fin[i][jn][v], vb = fin[i][jn][v + 1];
                const float send = odd ? va : vb;
                const float recv = __builtin_bit_cast(
                    float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, send), 0xB1, 0xF, 0xF, true));
                const bf16x2 pk = __builtin_convertvector((f32x2){odd ? recv : va, odd ? vb : recv}, bf16x2);
                if (pair && d < left_both) __builtin_memcpy(out + 2u * (both + (unsigned)(d * plane)), &pk, 4);
            }
        if (!pair)
#pragma unroll
            for (int i = 0; i < TF; ++i)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int d = i * 32 + (v >> 2) * 8 + (v & 3);
                    if (d < left)
                        *reinterpret_cast<unsigned short *>(out + 2u * (own + (unsigned)(d * plane))) = bf16_round(fin[i][jn][v]);
                }
    }
}

// One launch prepares both operands (layouts above).
//   blocks [0, xb_blocks): one thread per padded position of a channel block
//   the rest:              filters, one thread per 8-channel half
struct WindowPrepArgs {
    const unsigned short *src;
    u32x4 *xb;
    int64_t src_bs;
    int Cg, CBp;               // channels per column; its blocks, padded to whole chunks
    int LH, LW, Hp, Wp, pad_h, pad_w;
    unsigned positions;        // N * Hp * Wp
    unsigned total;            // groups * CBp * positions
    int xb_blocks;
    const unsigned short *w;
    u32x4 *wt;
    int M, Mpad, R, S, C, ncb; // C: channels per filter (the row stride of w)
    int transposed;            // backward-data: rows are the filter's channels, taps run backwards
    unsigned wt_halves;        // groups * CBp * R * S * Mpad * 2
    int64_t w_gs;
    FastDiv div_pos, div_hpwp, div_wp, div_cbp, div_mpad, div_ncb, div_taps;
};

__global__ __launch_bounds__(256) void window_prepare(const WindowPrepArgs p)
{
    unsigned short v[16];
    if ((int)blockIdx.x < p.xb_blocks) {
        const unsigned i = blockIdx.x * 256u + threadIdx.x;
        if (i >= p.total) return;
        const unsigned blk = fastdiv(i, p.div_pos), at = i - blk * p.positions;         // column's block; (n, hp, wp)
        const unsigned g = fastdiv(blk, p.div_cbp);
        const int c0 = (int)(blk - g * (unsigned)p.CBp) * 16;
        const unsigned n = fastdiv(at, p.div_hpwp), rem = at - n * (unsigned)(p.Hp * p.Wp);
        const int hp = (int)fastdiv(rem, p.div_wp), wp = (int)rem - hp * p.Wp;
        const int h = hp - p.pad_h, w = wp - p.pad_w, LHW = p.LH * p.LW;
        u32x4 lo = {0u, 0u, 0u, 0u}, hi = {0u, 0u, 0u, 0u};
        if ((unsigned)h < (unsigned)p.LH && (unsigned)w < (unsigned)p.LW && c0 < p.Cg) {    // Cg: whole blocks
            const unsigned short *const s = p.src + (int64_t)n * p.src_bs + (int64_t)((int)g * p.Cg + c0) * LHW + h * p.LW + w;
#pragma unroll
            for (int k = 0; k < 16; ++k) v[k] = s[(int64_t)k * LHW];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                lo[k] = (unsigned)v[2 * k] | ((unsigned)v[2 * k + 1] << 16);
                hi[k] = (unsigned)v[8 + 2 * k] | ((unsigned)v[8 + 2 * k + 1] << 16);
            }
        }
        const size_t swap = (at >> 3) & 1;
        p.xb[(size_t)i * 2 + swap] = lo;
        p.xb[(size_t)i * 2 + (swap ^ 1)] = hi;
        return;
    }
    const unsigned e = (blockIdx.x - (unsigned)p.xb_blocks) * 256u + threadIdx.x;
    if (e >= p.wt_halves) return;
    const unsigned t1 = e >> 1;                                        // (((g, chunk) taps + tap) ncb + b) Mpad + m
    const unsigned t2 = fastdiv(t1, p.div_mpad);
    const int m = (int)(t1 - t2 * (unsigned)p.Mpad);
    const unsigned t3 = fastdiv(t2, p.div_ncb), b = t2 - t3 * (unsigned)p.ncb;
    const unsigned gc = fastdiv(t3, p.div_taps);
    const int tap = (int)(t3 - gc * (unsigned)(p.R * p.S));
    const unsigned blk = gc * (unsigned)p.ncb + b, g = fastdiv(blk, p.div_cbp);
    const int ch0 = (int)(blk - g * (unsigned)p.CBp) * 16 + (int)(e & 1) * 8;
    const int rs = p.transposed ? p.R * p.S - 1 - tap : tap;
    const unsigned short *const w = p.w + (int64_t)g * p.w_gs;
    const bool ok = m < p.M && ch0 < p.Cg;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int ch = ch0 + k;
        v[k] = ok ? w[(p.transposed ? (int64_t)ch * p.C + m : (int64_t)m * p.C + ch) * (p.R * p.S) + rs] : (unsigned short)0;
    }
    const u32x4 o = {(unsigned)v[0] | ((unsigned)v[1] << 16), (unsigned)v[2] | ((unsigned)v[3] << 16),
                     (unsigned)v[4] | ((unsigned)v[5] << 16), (unsigned)v[6] | ((unsigned)v[7] << 16)};
    p.wt[(size_t)t1 * 2 + ((e & 1) ^ ((m >> 3) & 1))] = o;
}
