// Forward, backward-data and backward-filter of small problems (plan.h: direct) on the vector units, one launch a pass.
// Part of convnet_hotpath.hip: included there, inside its anonymous namespace, after the common definitions.
//
// Such a pass is a few microseconds of launches and of memory latency, not of arithmetic: the matrix kernels re-lay the
// filters in a launch of their own, pad few rows to 32 and run one serial chain of steps on a handful of work-groups.  Here
// the sixteen wavefronts of a work-group share the reduction, so that a chain is a sixteenth as long, read the tensors as
// they lie, and add their sums through LDS in a fixed order.  4 x 3 x 32 x 32, 16 filters 5x5: forward 9.8 -> 4.7 us,
// backward-data 25.3 -> 5.1, backward-filter 19.4 -> 6.0 (kernel times, launches of the old passes added up).

constexpr int kDirectWaves = 16, kDirectRows = 4;
constexpr int kWgradWaves = 8, kWgradFilters = 4;      // 75 work-groups of 16 wavefronts x 16 filters: 12.4 us
static_assert(kDirectRows == 4, "one 16-byte LDS read per reduction element");

struct DirectArgs {
    const void *w, *src;
    void *dst;
    int M, red;                // rows of the result; reduction length (channel, r, s)
    int S, RS, C;              // C: channels per filter
    int transposed;            // backward-data
    int OH, OW, LH, LW, stride, pad;
    int src_bs, dst_bs, ncols;
    int epi_on;
    Epilogue epi;
    FastDiv div_plane, div_ow, div_rs, div_s, div_stride;
};

// One work-group: POS positions x kDirectRows rows; its 1024 / POS groups of POS lanes share the reduction, eight loads at a
// time in flight (unconditional: a load under a condition is waited for before the next).  Taps and the rows' filters lie in
// LDS.  POS = 64 where that gives enough work-groups, else 16: a pass of 64 work-groups is bound by the instructions that
// sixteen wavefronts issue on one CU (backward-data above 12.6 us with POS = 64).
template <typename TI, typename TO, int POS>
__global__ __launch_bounds__(kDirectWaves * 64) void direct_colgemm_kernel(const DirectArgs p)
{
    constexpr int U = 8, PER_WAVE = 64 / POS, SLICES = kDirectWaves * PER_WAVE;
    // the element after the last is zero: what a group reads past its share, so that no infinity of another group's meets a zero
    __shared__ __attribute__((aligned(16))) float filt[(kDirectMaxRed + 1) * kDirectRows];
    __shared__ int2 taps[kDirectMaxRed + 1];                 // source plane, r << 16 | s
    __shared__ float sums[kDirectWaves][kDirectRows][POS];
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
    const int pos = lane % POS;
    const int m0 = blockIdx.y * kDirectRows;
    const int col = blockIdx.x * POS + pos;
    const int j = min(col, p.ncols - 1);
    const int n = (int)fastdiv((uint32_t)j, p.div_plane);
    const int rem = j - n * (p.OH * p.OW);
    const int oh = (int)fastdiv((uint32_t)rem, p.div_ow), ow = rem - oh * p.OW;
    const int hb = p.transposed ? oh + p.pad : oh * p.stride - p.pad, wb = p.transposed ? ow + p.pad : ow * p.stride - p.pad;
    const TI *const src = static_cast<const TI *>(p.src);
    const TI *const w = static_cast<const TI *>(p.w);

    for (int g = threadIdx.x; g < p.red; g += kDirectWaves * 64) {
        const int a = (int)fastdiv((uint32_t)g, p.div_rs), rs = g - a * p.RS;
        const int r = (int)fastdiv((uint32_t)rs, p.div_s), s = rs - r * p.S;
        taps[g] = make_int2(a * (p.LH * p.LW), p.transposed ? (-r << 16) | (-s & 0xffff) : r << 16 | s);
    }
    for (int i = threadIdx.x; i < p.red * kDirectRows; i += kDirectWaves * 64) {
        const int g = i / kDirectRows, m = min(m0 + i % kDirectRows, p.M - 1);
        const int a = (int)fastdiv((uint32_t)g, p.div_rs), rs = g - a * p.RS;
        filt[i] = ld_elem(w, p.transposed ? (int64_t)(a * p.C + m) * p.RS + rs : (int64_t)m * p.red + g);
    }
    if (threadIdx.x < kDirectRows) filt[p.red * kDirectRows + threadIdx.x] = 0.f;
    if (threadIdx.x == 0) taps[p.red] = make_int2(0, 0);
    __syncthreads();

    const int per = (p.red + SLICES - 1) / SLICES;
    const int g0 = (wave * PER_WAVE + lane / POS) * per;
    const int base = n * p.src_bs;
    float acc[kDirectRows] = {};
    const int g1 = min(g0 + per, p.red);
    for (int t = 0; t < per; t += U) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int g = g0 + t + u;
            const int2 tap = taps[g < g1 ? g : p.red];
            int h = hb + (tap.y >> 16), x = wb + (int)(short)tap.y;
            bool ok = g < g1;
            if (p.transposed && p.stride > 1) {
                const int hq = (int)fastdiv((uint32_t)max(h, 0), p.div_stride), xq = (int)fastdiv((uint32_t)max(x, 0), p.div_stride);
                ok = ok && hq * p.stride == h && xq * p.stride == x;
                h = hq; x = xq;
            }
            ok = ok && (unsigned)h < (unsigned)p.LH && (unsigned)x < (unsigned)p.LW;
            const float e = ld_elem(src, base + (ok ? tap.x + h * p.LW + x : 0));
            v[u] = ok ? e : 0.f;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int g = g0 + t + u;
            const f32x4 f = *reinterpret_cast<const f32x4 *>(&filt[(g < g1 ? g : p.red) * kDirectRows]);
#pragma unroll
            for (int i = 0; i < kDirectRows; ++i) acc[i] = fmaf(f[i], v[u], acc[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < kDirectRows; ++i) {
#pragma unroll
        for (int d = POS; d < 64; d *= 2) acc[i] += __shfl_xor(acc[i], d);
        if (lane < POS) sums[wave][i][lane] = acc[i];
    }
    __syncthreads();
    const int row_i = threadIdx.x / POS, q = threadIdx.x % POS;      // POS divides 64: lane's own position
    if (row_i < kDirectRows && col < p.ncols && m0 + row_i < p.M) {
        float v = sums[0][row_i][q];
#pragma unroll
        for (int i = 1; i < kDirectWaves; ++i) v += sums[i][row_i][q];
        const int row = m0 + row_i, plane = p.OH * p.OW;
        if (p.epi_on) v = epi_apply(p.epi, v, row, (int64_t)n * p.epi.mask_bs + (int64_t)row * plane + rem);
        st_elem(static_cast<TO *>(p.dst), (int64_t)n * p.dst_bs + (int64_t)row * plane + rem, v);
    }
}

struct DirectWgradArgs {
    const void *dy, *x;
    float *dw;
    int K, CRS, RS, S;
    int P, Q, H, W, stride, pad, dy_bs, x_bs, J;
    FastDiv div_plane, div_q, div_rs, div_s;
};

// One work-group: column (c, r, s) of dw for kWgradFilters filters, its threads over the positions.
template <typename TI>
__global__ __launch_bounds__(kWgradWaves * 64) void direct_wgrad_kernel(const DirectWgradArgs p)
{
    __shared__ float sums[kWgradWaves][kWgradFilters];
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
    const int g = blockIdx.x, k0 = blockIdx.y * kWgradFilters;
    const int c = (int)fastdiv((uint32_t)g, p.div_rs), rs = g - c * p.RS;
    const int r = (int)fastdiv((uint32_t)rs, p.div_s), s = rs - r * p.S;
    const int PQ = p.P * p.Q;
    const TI *const dy = static_cast<const TI *>(p.dy), *const x = static_cast<const TI *>(p.x);
    float acc[kWgradFilters] = {};
#pragma unroll 4
    for (int j = threadIdx.x; j < p.J; j += kWgradWaves * 64) {
        const int n = (int)fastdiv((uint32_t)j, p.div_plane);
        const int pq = j - n * PQ;
        const int pp = (int)fastdiv((uint32_t)pq, p.div_q);
        const int h = pp * p.stride - p.pad + r, w = (pq - pp * p.Q) * p.stride - p.pad + s;
        const bool ok = (unsigned)h < (unsigned)p.H && (unsigned)w < (unsigned)p.W;
        const float v = ld_elem(x, (int64_t)n * p.x_bs + (ok ? c * (p.H * p.W) + h * p.W + w : 0));
        float d[kWgradFilters];
#pragma unroll
        for (int k = 0; k < kWgradFilters; ++k) d[k] = ld_elem(dy, (int64_t)n * p.dy_bs + min(k0 + k, p.K - 1) * PQ + pq);
#pragma unroll
        for (int k = 0; k < kWgradFilters; ++k) acc[k] = fmaf(d[k], ok ? v : 0.f, acc[k]);
    }
    // four sums over 64 lanes: at each of two steps a lane keeps half of its sums and adds its partner's; then four steps over
    // the lanes that hold the same sum
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int keep = 2 >> b;
        const bool upper = lane & (1 << b);
#pragma unroll
        for (int k = 0; k < keep; ++k) {
            const float send = upper ? acc[k] : acc[k + keep], mine = upper ? acc[k + keep] : acc[k];
            acc[k] = mine + __shfl_xor(send, 1 << b);
        }
    }
#pragma unroll
    for (int d = 4; d < 64; d *= 2) acc[0] += __shfl_xor(acc[0], d);
    if (lane < 4) sums[wave][(lane & 1) * 2 + (lane >> 1)] = acc[0];
    __syncthreads();
    if (threadIdx.x < kWgradFilters && k0 + (int)threadIdx.x < p.K) {
        float v = sums[0][threadIdx.x];
#pragma unroll
        for (int i = 1; i < kWgradWaves; ++i) v += sums[i][threadIdx.x];
        p.dw[(int64_t)(k0 + threadIdx.x) * p.CRS + g] = v;
    }
}
