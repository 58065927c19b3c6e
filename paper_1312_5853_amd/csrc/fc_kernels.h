// Fully connected GEMM kernel, its split-sum kernel and the SGD update kernel.
// Part of convnet_hotpath.hip: included there, inside its anonymous namespace, after the common
// definitions (kThreads, kPitch, vector types); not a stand-alone header.
// ---------------------------------------------------------------------------
// Fully connected layers: D[M x Nc] = sum_k A(m, k) * B(k, n) on 128 x 128 tiles
// ---------------------------------------------------------------------------
//
// x [N][I], w [O][I], y [N][O], all row-major.  The three passes as GEMMs whose
// output has its columns contiguous in memory (so a wave's stores are 128-byte
// runs):
//   forward          y [N x O]  rows n, cols o, k = i:  A = x  (k contiguous),  B = w  (k contiguous)
//   backward-data    dx[N x I]  rows n, cols i, k = o:  A = dy (k contiguous),  B = w  (cols contiguous)
//   backward-filter  dw[O x I]  rows o, cols i, k = n:  A = dy (rows contiguous), B = x (cols contiguous)
// An operand with k contiguous ("k-major") is staged in LDS as [row][16] (pitch
// 20 floats) and read with b128 like the convolution tiles.  An operand whose
// rows / columns are contiguous ("transposed") is staged as [k][128] (pitch 132
// floats: 16-byte global loads become b128 LDS writes) and each lane reads its
// eight reduction elements with ds_read_b32: lanes 0..31 take consecutive
// floats, lanes 32..63 sit 8 * 132 floats further = 32 banks further, so both
// the writes and the reads are conflict-free.  Both operands feed reduction
// element 8 * (lane / 32) + t to the t-th matrix instruction of a step.
// Register sets, LDS double buffer and load / store slots between the matrix
// instructions work as in colgemm_fast_kernel.  The reduction is cut into
// ksplit ranges (grid = tiles * ksplit); with ksplit > 1 the kernel writes
// partial sums [ksplit][M][Nc] and fc_reduce_kernel adds them in a fixed order.
struct FcArgs {
    const float *A, *B;
    float *D;              // ksplit == 1: the result (row pitch ldd); else unused
    float *part;           // ksplit > 1: partial sums [ksplit][M][Nc]
    int M, Nc, K;
    int lda, ldb, ldd;
    int mtiles, ntiles, ksplit, steps_per_split;
    const float *bias;     // forward: one value per column (output neuron), or null
    int relu;
};

// A wave's sums (rows from m0, columns from n0): the result with bias and ReLU, or partial sums of range ks.  One 64-bit
// address, rows and column blocks at uniform distances from it; the blocks of a row one after the other, so that a row's 256
// bytes go out together (backward-filter 9216 -> 4096 at N = 2, bound by its 151 MB of stores: 37 us with a 64-bit product
// per store, 32.4 with the column blocks outside, 30.0 so; at N = 128 77, 75.1 and 73).
template <int TM, int TN>
__device__ __forceinline__ void fc_store_tile(const FcArgs &p, const f32x16 (&acc)[TM][TN], int ks, int m0, int n0, int lane)
{
    const int l32 = lane & 31, half = lane >> 5;
    // accumulator value v of block (i, jn): row 32 * i + 8 * (v / 4) + 4 * (lane / 32) + v % 4, column lane % 32
    const bool final_sums = p.ksplit == 1, relu = final_sums && p.relu;
    const int ldo = final_sums ? p.ldd : p.Nc, left = p.M - m0 - half * 4, right = p.Nc - n0 - l32;
    float *const out = (final_sums ? p.D : p.part + (size_t)ks * p.M * p.Nc) + (size_t)(m0 + half * 4) * ldo + n0 + l32;
    float bv[TN];
#pragma unroll
    for (int jn = 0; jn < TN; ++jn) {
        // The wait for the bias load must sit here, once: left to the compiler it lands in front of every
        // conditional store below, as a wait for ALL outstanding memory operations, the stores before it included,
        // so that the 64 stores of a tile went out one round trip at a time.
        bv[jn] = final_sums && p.bias && jn * 32 < right ? p.bias[n0 + jn * 32 + l32] : 0.f;
        asm volatile("" : "+v"(bv[jn]));          // the loaded value is complete from here on
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int d = i * 32 + (v >> 2) * 8 + (v & 3);
#pragma unroll
            for (int jn = 0; jn < TN; ++jn) {
                float r = acc[i][jn][v] + bv[jn];
                if (relu) r = r > 0.f ? r : 0.f;
                if (d < left && jn * 32 < right) out[(size_t)d * ldo + jn * 32] = r;
            }
        }
}

template <bool AT, bool BT>
__global__ __launch_bounds__(kThreads, 2) void fc_gemm_kernel(const FcArgs p)
{
    constexpr int TM = 2, TN = 2, BM = 128, BN = 128, KC = 16;
    constexpr int PK = KC + 4;                // [row][16] pitch
    constexpr int PT = 128 + 4;               // [k][128] pitch
    constexpr int ASZ = AT ? KC * PT : BM * PK, BSZ = BT ? KC * PT : BN * PK;
    __shared__ __attribute__((aligned(16))) float As0[2 * ASZ];
    __shared__ __attribute__((aligned(16))) float Bs0[2 * BSZ];

    const int ntile = p.mtiles * p.ntiles;
    const int unit = blockIdx.x;
    const int ks = unit / ntile;
    const int tile = unit - ks * ntile;
    const int mt = tile % p.mtiles, nt = tile / p.mtiles;
    const int m0 = mt * BM, n0 = nt * BN;
    const int k_begin = ks * p.steps_per_split * KC;
    const int k_end = min(p.K, k_begin + p.steps_per_split * KC);
    const int nsteps = (k_end - k_begin + KC - 1) / KC;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = uniform(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // Two 16-byte pieces per thread, operand and step.  k-major: piece q = tid + 256 * i covers row q / 4,
    // reduction elements 4 * (q % 4)..; transposed: reduction element q / 32, rows (columns) 4 * (q % 32)...
    // A piece outside the matrix or past the end of the reduction range reads the matrix base and stores zeros.
    const float *aptr[2], *bptr[2];
    int alds[2], blds[2], akoff[2], bkoff[2];
    bool arow[2], brow[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int q = tid + i * kThreads;
        if (AT) {
            const int k = q >> 5, c = (q & 31) * 4;
            arow[i] = m0 + c < p.M;
            akoff[i] = k;
            alds[i] = k * PT + c;
            aptr[i] = p.A + (size_t)(k_begin + k) * p.lda + (arow[i] ? m0 + c : 0);
        } else {
            const int row = q >> 2, kq = (q & 3) * 4;
            arow[i] = m0 + row < p.M;
            akoff[i] = kq;
            alds[i] = row * PK + kq;
            aptr[i] = p.A + (size_t)(arow[i] ? m0 + row : 0) * p.lda + k_begin + kq;
        }
        if (BT) {
            const int k = q >> 5, c = (q & 31) * 4;
            brow[i] = n0 + c < p.Nc;
            bkoff[i] = k;
            blds[i] = k * PT + c;
            bptr[i] = p.B + (size_t)(k_begin + k) * p.ldb + (brow[i] ? n0 + c : 0);
        } else {
            const int row = q >> 2, kq = (q & 3) * 4;
            brow[i] = n0 + row < p.Nc;
            bkoff[i] = kq;
            blds[i] = row * PK + kq;
            bptr[i] = p.B + (size_t)(brow[i] ? n0 + row : 0) * p.ldb + k_begin + kq;
        }
    }
    const size_t a_adv = AT ? (size_t)KC * p.lda : KC, b_adv = BT ? (size_t)KC * p.ldb : KC;

    f32x4 areg[2][2], breg[2][2];
    bool aok[2][2], bok[2][2];
    int kload = k_begin;                      // first reduction element of the next step to load
    auto slot_load = [&](int set, int q) {    // q = 0, 1: A pieces; 2, 3: B pieces (3 also advances the step)
        if (q < 2) {
            aok[set][q] = arow[q] && kload + akoff[q] < k_end;
            areg[set][q] = *reinterpret_cast<const f32x4 *>(aok[set][q] ? aptr[q] : p.A);
            aptr[q] += a_adv;
        } else {
            const int i = q - 2;
            bok[set][i] = brow[i] && kload + bkoff[i] < k_end;
            breg[set][i] = *reinterpret_cast<const f32x4 *>(bok[set][i] ? bptr[i] : p.B);
            bptr[i] += b_adv;
            if (i == 1) kload += KC;
        }
    };
    auto slot_store = [&](int set, int q) {   // the same pieces into LDS buffer `set`
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
        if (q < 2) *reinterpret_cast<f32x4 *>(&As0[set * ASZ + alds[q]]) = aok[set][q] ? areg[set][q] : zero;
        else *reinterpret_cast<f32x4 *>(&Bs0[set * BSZ + blds[q - 2]]) = bok[set][q - 2] ? breg[set][q - 2] : zero;
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int jn = 0; jn < TN; ++jn)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][jn][v] = 0.f;

    const int l32 = lane & 31, half = lane >> 5;
    const int a_frag = AT ? half * 8 * PT + wm * 64 + l32 : (wm * 64 + l32) * PK + half * 8;
    const int b_frag = BT ? half * 8 * PT + wn * 64 + l32 : (wn * 64 + l32) * PK + half * 8;
    constexpr int NMMA = 8 * TM * TN;

    if (nsteps > 0) {
#pragma unroll
        for (int q = 0; q < 4; ++q) slot_load(0, q);
#pragma unroll
        for (int q = 0; q < 4; ++q) slot_store(0, q);
        if (nsteps > 1) {
#pragma unroll
            for (int q = 0; q < 4; ++q) slot_load(1, q);
        }
    }
    __syncthreads();

    // par / mode as in colgemm_fast_kernel: mode 2 = loads of step + 2 and stores of step + 1, 1 = stores only
    auto do_step = [&](auto par_c, auto mode_c) {
        constexpr int par = decltype(par_c)::value, mode = decltype(mode_c)::value;
        const float *As = As0 + par * ASZ, *Bs = Bs0 + par * BSZ;
        float fa[TM][8], fb[TN][8];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            if (AT) {
#pragma unroll
                for (int t = 0; t < 8; ++t) fa[i][t] = As[a_frag + t * PT + i * 32];
            } else {
                const f32x4 *q = reinterpret_cast<const f32x4 *>(&As[a_frag + i * 32 * PK]);
                const f32x4 lo = q[0], hi = q[1];
#pragma unroll
                for (int t = 0; t < 4; ++t) { fa[i][t] = lo[t]; fa[i][4 + t] = hi[t]; }
            }
        }
#pragma unroll
        for (int jn = 0; jn < TN; ++jn) {
            if (BT) {
#pragma unroll
                for (int t = 0; t < 8; ++t) fb[jn][t] = Bs[b_frag + t * PT + jn * 32];
            } else {
                const f32x4 *q = reinterpret_cast<const f32x4 *>(&Bs[b_frag + jn * 32 * PK]);
                const f32x4 lo = q[0], hi = q[1];
#pragma unroll
                for (int t = 0; t < 4; ++t) { fb[jn][t] = lo[t]; fb[jn][4 + t] = hi[t]; }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < NMMA; ++m) {
            const int t = m / (TM * TN), i = (m / TN) % TM, jn = m % TN;
            acc[i][jn] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][t], fb[jn][t], acc[i][jn], 0, 0, 0);
            if (mode > 0 && m < 8) {          // one slot after each of the first eight matrix instructions
                __builtin_amdgcn_sched_barrier(0);
                if (m < 4) {
                    if (mode == 2) slot_load(par, m);
                } else {
                    slot_store(par ^ 1, m - 4);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (mode > 0) __syncthreads();
    };
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    using M2 = std::integral_constant<int, 2>;
    int step = 0;
    for (; step + 3 < nsteps; step += 2) {
        do_step(P0{}, M2{});
        do_step(P1{}, M2{});
    }
    const int rest = nsteps - step;
    if (rest == 3) {
        do_step(P0{}, M2{});
        do_step(P1{}, P1{});
        do_step(P0{}, P0{});
    } else if (rest == 2) {
        do_step(P0{}, P1{});
        do_step(P1{}, P0{});
    } else if (rest == 1) {
        do_step(P0{}, P0{});
    }

    fc_store_tile<TM, TN>(p, acc, ks, m0 + wm * TM * 32, n0 + wn * TN * 32, lane);
}

// ---------------------------------------------------------------------------
// The same GEMMs on the bf16 matrix instruction, operands split into three bfloat16 parts in registers (six products, two
// accumulators: arithmetic, error and range as in conv_split_kernels.h).  A weight is read once, in fp32, and split once per
// row tile: a split copy in memory would cost more than the whole pass.
// Same tiles, ranges and partial sums as fc_gemm_kernel; four waves of 64 x 64, two work-groups per CU, so that one's
// stores pass under the other's matrix instructions (backward-filter has only N / 16 steps per tile).
// A staged piece is eight values of one row at consecutive k (operand with k contiguous) or of eight consecutive rows at
// one k (transposed), loaded as two 16-byte quads two steps ahead, split and stored between the matrix instructions.
// LDS, per part and 16-deep step, 32 bytes per line:
//   k contiguous  [128 rows][16 k]: lower half k = 0..7, upper half k = 12..15, 8..11, halves swapped where (row >> 3) & 1
//   transposed    [8 blocks of 16 rows][16 k]: k in line k ^ 4 * (block & 1), read with ds_read_b64_tr_b16 (the order of k
//                 inside a fragment is the one above, see conv_wgrad_split_kernels.h)
// Raw buffer loads read zero outside the matrices and past the range: tensors of 2^31 bytes and more go to fc_gemm_kernel.
// 9216 -> 4096, N = 128, kernel and sum of the partials: forward 101 -> 69 us, backward-data 106 -> 67, backward-filter
// 113 -> 73; error against 64 bits 4.4e-7 -> 1.5e-7.  Bound: matrix instructions 45 % of the time at one barrier per 16-deep
// step; of the backward-filter the first loads of each tile's short reduction and the 151 MB it writes.
// ---------------------------------------------------------------------------
template <bool AT, bool BT>
__global__ __launch_bounds__(kThreads, 2) void fc_split_kernel(const FcArgs p)
{
    constexpr int TM = 2, TN = 2, BM = 128, BN = 128, KC = 16;
    constexpr int PART = 4096, BUF = 6 * PART;                 // bytes: one part of one operand; both operands of a step
    constexpr int MPG = TM * TN;
    constexpr unsigned kOutside = 0x80000000u;
    __shared__ __attribute__((aligned(16))) char tiles[2 * BUF];

    const int ntile = p.mtiles * p.ntiles;
    const int unit = blockIdx.x;
    const int ks = unit / ntile;
    const int tile = unit - ks * ntile;
    const int mt = tile % p.mtiles, nt = tile / p.mtiles;
    const int m0 = mt * BM, n0 = nt * BN;
    const int k_begin = ks * p.steps_per_split * KC;
    const int k_end = min(p.K, k_begin + p.steps_per_split * KC);
    const int nsteps = (k_end - k_begin + KC - 1) / KC;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = uniform(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // bytes of the operands (below 2^31): rows x pitch
    const int a_bytes = (AT ? p.K : p.M) * p.lda * 4, b_bytes = (BT ? p.K : p.Nc) * p.ldb * 4;
    const auto rsrc_a = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.A), 0, a_bytes, 0x00020000);
    const auto rsrc_b = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p.B), 0, b_bytes, 0x00020000);

    // Offsets of this lane's two quads (relative to step 0 of the range), the k at which each ends being inside, LDS address
    struct Piece { unsigned off[2], lds; int k[2]; };
    auto make_piece = [&](bool transposed, int row0, int rows, int ld) {
        Piece q;
        if (transposed) {
            const int k = wave * 4 + ((lane >> 1) & 3), b = lane >> 3, o = lane & 1;
            const int r = row0 + b * 16 + o * 8;
            q.lds = (unsigned)(b * 512 + (k ^ ((b & 1) * 4)) * 32 + o * 16);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                q.off[h] = r + 4 * h < rows ? ((unsigned)(k_begin + k) * (unsigned)ld + (unsigned)(r + 4 * h)) * 4u : kOutside;
                q.k[h] = k;
            }
        } else {
            const int row = wave * 32 + (lane >> 1), o = lane & 1;
            q.lds = (unsigned)(row * 32 + (o ^ ((row >> 3) & 1)) * 16);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                q.k[h] = o ? 12 - 4 * h : 4 * h;
                q.off[h] = row0 + row < rows ? ((unsigned)(row0 + row) * (unsigned)ld + (unsigned)(k_begin + q.k[h])) * 4u : kOutside;
            }
        }
        return q;
    };
    const Piece pc[2] = {make_piece(AT, m0, p.M, p.lda), make_piece(BT, n0, p.Nc, p.ldb)};
    const unsigned adv[2] = {(unsigned)(AT ? KC * p.lda : KC) * 4u, (unsigned)(BT ? KC * p.ldb : KC) * 4u};

    f32x4 st[2][2][2];                          // [set][operand][quad]: step t is in set t & 1
    int kload = k_begin;                        // first k of the next step to load
    unsigned moved[2] = {0u, 0u};               // bytes since step 0
    auto load_quad = [&](int set, int op, int h) {
        unsigned v = pc[op].off[h], moved_op = moved[op];
        if (kload + KC > k_end) {                // (uniform) the range ends in this step, or has ended: nothing is read then
            v = kload + pc[op].k[h] < k_end ? v : kOutside;
            moved_op = kload < k_end ? moved_op : 0u;
        }
        st[set][op][h] = __builtin_bit_cast(f32x4, op == 0 ? __builtin_amdgcn_raw_buffer_load_b128(rsrc_a, v, moved_op, 0)
                                                           : __builtin_amdgcn_raw_buffer_load_b128(rsrc_b, v, moved_op, 0));
    };
    auto next_load_step = [&]() { kload += KC; moved[0] += adv[0]; moved[1] += adv[1]; };
    u32x4 sp[3];
    auto split_two = [&](int set, int op, int t) {
        unsigned h, m, l;
        split_pair(st[set][op][t >> 1][2 * (t & 1)], st[set][op][t >> 1][2 * (t & 1) + 1], h, m, l);
        sp[0][t] = h; sp[1][t] = m; sp[2][t] = l;
    };
    auto store_piece = [&](int buf, int op) {
        char *const d = tiles + buf * BUF + op * 3 * PART + pc[op].lds;
#pragma unroll
        for (int c = 0; c < 3; ++c) *reinterpret_cast<u32x4 *>(d + c * PART) = sp[c];
    };

    f32x16 acc[TM][TN], low[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int jn = 0; jn < TN; ++jn)
#pragma unroll
            for (int v = 0; v < 16; ++v) { acc[i][jn][v] = 0.f; low[i][jn][v] = 0.f; }

    // fragment of 32 rows: one 16-byte read, or two transposing reads of four k each
    const int l32 = lane & 31, half = lane >> 5;
    const int sub = (lane >> 4) & 1;
    const unsigned straight = (unsigned)(l32 * 32 + (half ^ ((l32 >> 3) & 1)) * 16);
    const unsigned across = (unsigned)(sub * 512 + (((half ? 12 : 0) ^ (sub * 4)) + ((lane & 15) >> 2)) * 32 + (lane & 3) * 8);
    typedef __attribute__((address_space(3))) char *lds_bytes;
    typedef __attribute__((address_space(3))) s16x4 *lds_quad;
    typedef short s16x8 __attribute__((ext_vector_type(8)));
    const lds_bytes at_lo = (lds_bytes)tiles + across, at_hi = (lds_bytes)tiles + (across ^ 128u);
    auto read_frag = [&](bool transposed, int off) {
        if (transposed) {
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad)(at_lo + off));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_quad)(at_hi + off));
            return (s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
        return *reinterpret_cast<const s16x8 *>(tiles + straight + off);
    };
    s16x8 fa[3][TM], fb[3][TN];
    auto read_a = [&](int buf, int c) {
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[c][i] = read_frag(AT, buf * BUF + c * PART + (wm * TM + i) * 1024);
    };
    auto read_b = [&](int buf, int c) {
#pragma unroll
        for (int jn = 0; jn < TN; ++jn) fb[c][jn] = read_frag(BT, buf * BUF + (3 + c) * PART + (wn * TN + jn) * 1024);
    };

#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int q = 0; q < 4; ++q) load_quad(t, q >> 1, q & 1);
        next_load_step();
    }
#pragma unroll
    for (int op = 0; op < 2; ++op) {
#pragma unroll
        for (int t = 0; t < 4; ++t) split_two(0, op, t);
        store_piece(0, op);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) load_quad(0, q >> 1, q & 1);
    next_load_step();
    __syncthreads();
    read_a(0, 0);
    read_b(0, 0);

    // One step out of buffer `par`: the pieces of step + 1 (set par ^ 1) are split and stored and those of step + 3 loaded
    // into their registers ahead of the barrier; the last two products cover it and the next step's first reads.
    auto do_step = [&](auto par_c) {
        constexpr int par = decltype(par_c)::value, oth = par ^ 1;
        auto work = [&](auto i_c) {              // 7 per operand: S0 S1 L0 S2 S3 store L1
            constexpr int op = decltype(i_c)::value / 7, s = decltype(i_c)::value % 7;
            if constexpr (op < 2) {
                if constexpr (s == 2) load_quad(oth, op, 0);
                else if constexpr (s == 5) store_piece(oth, op);
                else if constexpr (s == 6) load_quad(oth, op, 1);
                else split_two(oth, op, s < 2 ? s : s - 1);
            }
        };
        auto product = [&](auto ca_c, auto cb_c, auto g_c) {
            constexpr int ca = decltype(ca_c)::value, cb = decltype(cb_c)::value, g = decltype(g_c)::value;
            static_for<MPG>([&](auto q_c) {
                constexpr int i = decltype(q_c)::value / TN, jn = decltype(q_c)::value % TN, m = g * MPG + decltype(q_c)::value;
                f32x16 &sum = g == 0 ? acc[i][jn] : low[i][jn];
                sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa[ca][i]),
                                                              __builtin_bit_cast(bf16x8, fb[cb][jn]), sum, 0, 0, 0);
                if constexpr (m < 14) {
                    __builtin_amdgcn_sched_barrier(0);
                    work(I<m>{});
                    __builtin_amdgcn_sched_barrier(0);
                }
            });
            __builtin_amdgcn_sched_barrier(0);
        };
        read_b(par, 2);
        read_a(par, 2);
        __builtin_amdgcn_sched_barrier(0);
        product(I<0>{}, I<0>{}, I<0>{});
        read_b(par, 1);
        read_a(par, 1);
        __builtin_amdgcn_sched_barrier(0);
        product(I<0>{}, I<2>{}, I<1>{});
        product(I<2>{}, I<0>{}, I<2>{});
        product(I<0>{}, I<1>{}, I<3>{});
        asm volatile("s_waitcnt lgkmcnt(0)");
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        read_a(oth, 0);
        __builtin_amdgcn_sched_barrier(0);
        product(I<1>{}, I<0>{}, I<4>{});
        next_load_step();
        read_b(oth, 0);
        __builtin_amdgcn_sched_barrier(0);
        product(I<1>{}, I<1>{}, I<5>{});
    };
    for (int step = 0; step < nsteps; step += 2) {
        do_step(I<0>{});
        if (step + 1 < nsteps) do_step(I<1>{});
    }

    // sums that call for fp32 arithmetic: the whole work-group computes its tile again
    {
        bool col_ok[TN];
#pragma unroll
        for (int jn = 0; jn < TN; ++jn) col_ok[jn] = n0 + (wn * TN + jn) * 32 + l32 < p.Nc;
        auto scan = [&](int *nan_rows, int *nan_cols) {
            kload = k_begin;
            moved[0] = moved[1] = 0u;
#pragma unroll 1
            for (int step = 0; step < nsteps; ++step) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const bool across_k = q < 2 ? AT : BT;           // four rows at one k, or four k of one row
                    int *const mark = (q < 2 ? nan_rows : nan_cols) +
                                      (across_k ? (lane >> 3) * 16 + (lane & 1) * 8 + (q & 1) * 4 : wave * 32 + (lane >> 1));
                    load_quad(0, q >> 1, q & 1);
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        if (is_nan_bits(__float_as_uint(st[0][q >> 1][q & 1][t]))) mark[across_k ? t : 0] = 1;
                }
                next_load_step();
            }
        };
        if (split_finish<TM, TN, 4, BM, BN>(acc, low, wm * TM * 32 + half * 4, p.M - m0, wn * TN * 32 + l32, col_ok,
                                            reinterpret_cast<int *>(tiles), wave, lane, scan)) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int jn = 0; jn < TN; ++jn)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][jn][v] = 0.f;
#pragma unroll 1
            for (int k0 = k_begin; k0 < k_end; k0 += 8) {        // the loads of eight elements in flight, unconditional
                float a[4][TM], b[4][TN];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int k = k0 + t * 2 + half, kc = min(k, k_end - 1);
#pragma unroll
                    for (int i = 0; i < TM; ++i) {
                        const int r = m0 + (wm * TM + i) * 32 + l32, rc = min(r, p.M - 1);
                        const float e = p.A[AT ? (size_t)kc * p.lda + rc : (size_t)rc * p.lda + kc];
                        a[t][i] = k < k_end && r < p.M ? e : 0.f;
                    }
#pragma unroll
                    for (int jn = 0; jn < TN; ++jn) {
                        const int r = n0 + (wn * TN + jn) * 32 + l32, rc = min(r, p.Nc - 1);
                        const float e = p.B[BT ? (size_t)kc * p.ldb + rc : (size_t)rc * p.ldb + kc];
                        b[t][jn] = k < k_end && r < p.Nc ? e : 0.f;
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
    fc_store_tile<TM, TN>(p, acc, ks, m0 + wm * TM * 32, n0 + wn * TN * 32, lane);
}

// D[m][n] = part[0][m][n] + part[1][m][n] + ... (fixed order), then bias per column and ReLU.  Four columns per thread
// (Nc is a multiple of four), the loads of eight partials in flight.
__global__ __launch_bounds__(256) void fc_reduce_kernel(const float *__restrict__ part, float *__restrict__ D, int nsplit,
                                                        int M, int Nc, int ldd, const float *__restrict__ bias, int relu)
{
    const int64_t quads = (int64_t)M * Nc / 4;
    const f32x4 *src = reinterpret_cast<const f32x4 *>(part);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < quads; i += (int64_t)gridDim.x * blockDim.x) {
        f32x4 v = src[i];
#pragma unroll 8
        for (int k = 1; k < nsplit; ++k) v += src[(size_t)k * quads + i];
        const int m = (int)(i * 4 / Nc), n = (int)(i * 4 - (int64_t)m * Nc);
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (bias) v[t] += bias[n + t];
            if (relu) v[t] = v[t] > 0.f ? v[t] : 0.f;
        }
        *reinterpret_cast<f32x4 *>(D + (size_t)m * ldd + n) = v;
    }
}

// The same update for up to kSgdMaxTensors parameter tensors in ONE launch: tensor t owns the blocks
// [first_block[t], first_block[t + 1]) of 256 threads x 4 parameters (16-byte aligned tensors) or x 1 parameter.
constexpr int kSgdMaxTensors = 24;
struct SgdMultiArgs {
    float *w[kSgdMaxTensors];
    const float *dw[kSgdMaxTensors];
    float *vel[kSgdMaxTensors];
    int64_t count[kSgdMaxTensors];
    unsigned first_block[kSgdMaxTensors + 1];
    int vec[kSgdMaxTensors];
    int n;
    float lr, momentum, weight_decay, grad_scale;
};

__device__ __forceinline__ void sgd_update_elems(float *__restrict__ w, const float *__restrict__ dw,
                                                 float *__restrict__ vel, int64_t count, int64_t i, float lr,
                                                 float momentum, float weight_decay, float grad_scale, int vec);

__global__ void sgd_update_multi_kernel(const SgdMultiArgs a)
{
    int t = 0;
    while (t + 1 < a.n && blockIdx.x >= a.first_block[t + 1]) ++t;          // uniform: at most 23 steps
    const int64_t i = (int64_t)(blockIdx.x - a.first_block[t]) * blockDim.x + threadIdx.x;
    sgd_update_elems(a.w[t], a.dw[t], a.vel[t], a.count[t], i, a.lr, a.momentum, a.weight_decay, a.grad_scale, a.vec[t]);
}

// SGD with momentum and weight decay, one thread per four parameters:
//   v = momentum * v - lr * (weight_decay * w + grad_scale * dw);  w += v
__device__ __forceinline__ void sgd_update_elems(float *__restrict__ w, const float *__restrict__ dw,
                                                 float *__restrict__ vel, int64_t count, int64_t i, float lr,
                                                 float momentum, float weight_decay, float grad_scale, int vec)
{
    if (vec) {
        const int64_t n4 = count >> 2;
        if (i < n4) {
            f32x4 wv = reinterpret_cast<f32x4 *>(w)[i];
            const f32x4 g = reinterpret_cast<const f32x4 *>(dw)[i];
            f32x4 v = reinterpret_cast<f32x4 *>(vel)[i];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = momentum * v[e] - lr * (weight_decay * wv[e] + grad_scale * g[e]);
                wv[e] += v[e];
            }
            reinterpret_cast<f32x4 *>(vel)[i] = v;
            reinterpret_cast<f32x4 *>(w)[i] = wv;
        }
        const int64_t t = (n4 << 2) + i;      // scalar tail
        if (i < (count & 3)) {
            const float v = momentum * vel[t] - lr * (weight_decay * w[t] + grad_scale * dw[t]);
            vel[t] = v;
            w[t] += v;
        }
    } else if (i < count) {
        const float v = momentum * vel[i] - lr * (weight_decay * w[i] + grad_scale * dw[i]);
        vel[i] = v;
        w[i] += v;
    }
}

__global__ void sgd_update_kernel(float *__restrict__ w, const float *__restrict__ dw, float *__restrict__ vel,
                                  int64_t count, float lr, float momentum, float weight_decay, float grad_scale,
                                  int vec)
{
    sgd_update_elems(w, dw, vel, count, (int64_t)blockIdx.x * blockDim.x + threadIdx.x, lr, momentum, weight_decay,
                     grad_scale, vec);
}
