// fp32 forward / stride-1 backward-data on the 16-bit matrix instructions: every fp32 operand is split into three bfloat16
// parts whose sum it is, and the six products that matter are accumulated in fp32; or, for long sums of operands of like
// magnitudes, into two half-precision parts and three products (see operand_range below).
// Part of convnet_hotpath.hip: included there, inside its anonymous namespace, after conv_bf16_dma_kernels.h.
//
// Why: an fp32 matrix instruction occupies the pipe 16 times as long per product as a bf16 one.  x = h + m + l with
// h = bf16(x), m = bf16(x - h), l = x - h - m is exact (8 + 8 + 8 significand bits, every remainder representable), so
//   x * w = h h' + h m' + m h' + m m' + h l' + l h'  (+ m l' + l m' + l l', at most 2^-24 |x w|, random in sign, left out)
// costs six bf16 products: 16 / 6 = 2.7 times the fp32 rate.  The matrix instruction adds its 16 products to the fp32
// accumulator with one rounding (v_mfma_f32_32x32x2_f32: eight per 16 products); h h' has an accumulator of its own, the
// five smaller products, whose roundings weigh 2^-8 as much, share another, and the two are added at the end.  Relative
// error (2-norm) against 64-bit sums, 384 channels 3x3 forward: 2.7e-7; fp32 kernel 6.7e-7; with one accumulator for all
// six products 8.1e-7.
//
// Range: each operand is split as 2^24 times itself and a sum is multiplied by 2^-48 at the end, both exact, so that the parts
// of every finite fp32 value below 2^104, subnormal ones included, are zero or normal bfloat16 numbers: small operands keep
// all their bits, whatever lies beside them or multiplies them.  What no longer fits, operands from 2^104 and sums from 2^80
// on, makes its sum infinite or NaN, and the work-group computes such a tile again from the fp32 tensors with the fp32 matrix
// instruction (split_finish), so that large values, infinities and NaN come out as fp32 arithmetic gives them.

template <int V> using I = std::integral_constant<int, V>;
template <typename F, int... V>
__device__ __forceinline__ void static_for_seq(F &&f, std::integer_sequence<int, V...>) { (f(I<V>{}), ...); }
template <int N, typename F> __device__ __forceinline__ void static_for(F &&f)
{
    static_for_seq(f, std::make_integer_sequence<int, N>{});
}

constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f;

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// two fp32 values -> the bfloat16 parts of 2^24 times them, two to a word
__device__ __forceinline__ void split_pair(float a, float b, unsigned &h, unsigned &m, unsigned &l)
{
    a *= kSplitScale;
    b *= kSplitScale;
    h = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){a, b}, bf16x2));
    const float a1 = a - __uint_as_float(h << 16), b1 = b - __uint_as_float(h & 0xffff0000u);
    m = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){a1, b1}, bf16x2));
    const float a2 = a1 - __uint_as_float(m << 16), b2 = b1 - __uint_as_float(m & 0xffff0000u);
    l = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){a2, b2}, bf16x2));
}

// eight consecutive reduction elements -> one 16-byte piece of each part
__device__ __forceinline__ void split_eight(const float (&v)[8], u32x4 (&o)[3])
{
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        unsigned h, m, l;
        split_pair(v[2 * t], v[2 * t + 1], h, m, l);
        o[0][t] = h; o[1][t] = m; o[2][t] = l;
    }
}

// ---------------------------------------------------------------------------
// Two half-precision parts: h = f16(s x), l = f16((s x - h) 2^12), s a power of two that brings the largest operand of the
// tensor into [2^14, 2^15).  s x = h + 2^-12 l up to 2^-23 of itself (11 + 11 significand bits and l's sign) where the operand is
// within 2^-28 of the largest, 2^-20 at 2^-32 of it; three products, h h' into one accumulator, h l' and l h' into another.  A
// call takes them where, in both tensors, every operand is zero or within these 2^-32, nearly all of them (kMostTiny) within 2^-27,
// the largest lie between 2^-45 and 2^41, and magnitudes spread far enough (kLeastFine); any other call, and so every one with an
// infinity, a NaN or a value whose products could leave fp32's range, keeps the three bfloat16 parts.  operand_range looks at the
// tensors, on the GPU, and the kernels branch on what it found.
// ---------------------------------------------------------------------------
constexpr int kRangeBlocks = 256, kRangeThreads = 512;       // per tensor
// The largest operand of a tensor may lie 2^7 above the mean magnitude of its sample (in normal, uniform and Laplace draws of 2^23 it
// lies 2^5 above), and a share of 2^-14 of the operands, less than a sample, a channel or a filter, 2^-20 below it: the others are
// within 2^-27 of the largest, which two parts hold in 23 bits.  Errors against 64 bits of two parts and three: both tensors 2^-31
// to 2^-29 below one operand, sums of 2304, 1.4e-7 and 7.1e-8; filters exp(2 z) of normal z, sums of 864, few products that
// decide, 2.2e-7 and 1.7e-7.
constexpr int kMostAbove = 7;
constexpr unsigned kTinyBinades = 20;
constexpr float kMostTiny = 0x1p-14f;
// The sums of h h' of bfloat16 parts stay exact, and theirs is the smaller error, while every product is a multiple of the sum's
// last bit: where magnitudes lie within few binades, or have few bits.  An operand is fine below an eighth of the mean magnitude
// of its tensor's sample; c: the share of products with a fine operand.  Errors of two parts over those of three, sums of 54 to 300
// steps, of c: both tensors' magnitudes in [0.25, 1) 0: 4.4; in [1/16, 1) 0.01: 1.34; [0.5, 1) by a normal tensor 0.08: 1.13; mean
// of 3 deviations by normal 0.083: 1.09; of 2 deviations 0.105: 1.02 to 1.04; 95 % in [0.5, 1), 5 % about 0.01, by normal 0.126:
// 0.97 to 1.01; uniform by normal 0.138: 0.80 to 0.93; normal by normal 0.153: 0.80 to 0.94; Laplace 0.22: 0.76 to 0.86.  And three
// parts compute where most of the sample's fine operands end, in bfloat16, in two zero bits (8-bit integers by normal: 1.30).
constexpr float kFineShare = 0.125f, kLeastFine = 0.129f;
constexpr float kHalfLow = 0x1p12f, kHalfLowInv = 0x1p-12f;

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

// What the kernels of a call read in memory, for each column of a grouped layer: what each block of operand_range found of its part
// of each tensor, and what follows.
struct SplitInfo {
    int segments;              // two parts, the sums of h h' in so many segments; or 0: three parts
    float unscale;             // of a sum
    float sa, sb;              // of the tensors' operands
};
struct SplitRanges {
    unsigned ends[2][kRangeBlocks];          // exponent of the largest, 255 less that of the smallest that is not zero, tiny ones
    unsigned zeros[2][kRangeBlocks];         // and whether any is negative, the highest bit
    unsigned fine[2][kRangeBlocks];
    float operand[2];                        // one as a share of all
    int most_big[2];                         // the exponent that the largest may have
    int few_bits[2];                         // most of the sample's fine operands have few bits
    int none;                                // nothing was looked at
    SplitInfo info;                          // by the preparation
};

struct RangeArgs {
    const float *t[2];
    unsigned bs[2];            // elements between samples (tensors have less than 2^29)
    int64_t gs[2];             // elements between columns
    unsigned len[2], quads[2]; // elements of a sample (four and more), its groups of four
    unsigned total[2];         // groups of four in all
    FastDiv div_quads[2];
    int signed_only;           // three parts where tensor 0 has no negative operand
    int steps;                 // see split_segments
    float dense;
    SplitRanges *out;
};

template <int CTRL> __device__ __forceinline__ unsigned dpp(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xf, 0xf, false);
}
// largest (smallest) value over a wavefront whose lanes are all active
__device__ __forceinline__ unsigned wave_max(unsigned v)
{
    v = max(v, dpp<0x111>(v)); v = max(v, dpp<0x112>(v)); v = max(v, dpp<0x114>(v)); v = max(v, dpp<0x118>(v));
    v = max(v, dpp<0x142>(v)); v = max(v, dpp<0x143>(v));
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ __forceinline__ unsigned wave_min(unsigned v) { return ~wave_max(~v); }
template <int CTRL, int ROWS> __device__ __forceinline__ unsigned dpp_or_zero(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ unsigned wave_sum(unsigned v)
{
    v += dpp_or_zero<0x111, 0xf>(v); v += dpp_or_zero<0x112, 0xf>(v); v += dpp_or_zero<0x114, 0xf>(v); v += dpp_or_zero<0x118, 0xf>(v);
    v += dpp_or_zero<0x142, 0xa>(v); v += dpp_or_zero<0x143, 0xc>(v);
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}
// over lanes 0 to 31 in lane 31, over lanes 32 to 63 in lane 63
__device__ __forceinline__ unsigned half_max(unsigned v)
{
    v = max(v, dpp<0x111>(v)); v = max(v, dpp<0x112>(v)); v = max(v, dpp<0x114>(v)); v = max(v, dpp<0x118>(v));
    return max(v, dpp_or_zero<0x142, 0xa>(v));
}
__device__ __forceinline__ unsigned half_sum(unsigned v)
{
    v += dpp_or_zero<0x111, 0xf>(v); v += dpp_or_zero<0x112, 0xf>(v); v += dpp_or_zero<0x114, 0xf>(v); v += dpp_or_zero<0x118, 0xf>(v);
    return v + dpp_or_zero<0x142, 0xa>(v);
}
template <int CTRL, int ROWS> __device__ __forceinline__ float dpp_or_zero(float v)
{
    return __uint_as_float(dpp_or_zero<CTRL, ROWS>(__float_as_uint(v)));
}
__device__ __forceinline__ float wave_sum(float v)
{
    v += dpp_or_zero<0x111, 0xf>(v); v += dpp_or_zero<0x112, 0xf>(v); v += dpp_or_zero<0x114, 0xf>(v); v += dpp_or_zero<0x118, 0xf>(v);
    v += dpp_or_zero<0x142, 0xa>(v); v += dpp_or_zero<0x143, 0xc>(v);
    return __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(v), 63));
}

// A forward pass keeps three parts for an input of one sign (the output of a ReLU or of pooling): for such inputs the error of
// two is the smaller one by 5 to 25 % only, and a pooling window behind the layer, or a ReLU, that decides between values closer
// than a rounding sends a gradient elsewhere, so that another rounding of a network's forward pass, however small its errors, moves
// its gradients by 1e-3 either way.
// Bound: HBM, four bytes per operand; every operand is read once here and once by what follows, from the 256 MB cache where the
// tensors fit.  A group of four that would reach past a sample's end is moved back: operands seen twice change nothing.
// 128 x 384 x 13 x 13 and its filters 10.8 us, with as large a gradient 14.6, ended by the sample 5.2; two columns of 128 x 48 x 27 x 27
// and 128 x 128 x 27 x 27 21.5 a pass in the mean (one look for both 19.8; four groups of a thread in flight instead of two 21.9).
// A column of a grouped layer (blockIdx.y) is looked at by itself, so that it takes the parts that it takes in a call of its own.
__global__ __launch_bounds__(kRangeThreads, 8) void operand_range(const RangeArgs p)
{
    typedef unsigned quad_t __attribute__((ext_vector_type(4), aligned(4)));
    const int which = (int)blockIdx.x >= kRangeBlocks, b = (int)blockIdx.x - which * kRangeBlocks;
    const float *const t = p.t[which] + blockIdx.y * p.gs[which];
    SplitRanges *const out = p.out + blockIdx.y;
    const unsigned total = p.total[which];
    // element that group q of tensor u begins with
    const auto place_of = [&](int u, unsigned q) {
        const unsigned n = fastdiv(q, p.div_quads[u]);
        return n * p.bs[u] + min((q - n * p.quads[u]) * 4, p.len[u] - 4);
    };
    // Every block looks at the same 2048 operands of each tensor first, sixteen at each of 128 places, one in each 128th of the
    // tensor at a distance from its start that is another in each (with one distance, places fall on the same rows of a channel
    // in sample after sample): where these say that three parts are to compute, that is all.
    __shared__ unsigned words[6][kRangeThreads / 64];
    unsigned tiny_line, fine_line;                               // of this block's tensor; operands less one below are tiny / fine
    {
        unsigned none = 0, negative = 0;                         // zeros of tensor 0, + 2^16 of tensor 1
        float sum = 0.f;                                         // of the magnitudes of this block's tensor
        quad_t mine;                                             // its operands of this thread
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const unsigned place = threadIdx.x >> 2, share = p.total[u] / (kRangeThreads / 4);
            const unsigned q = min(place * share + __umulhi(place * 0x9e3779b9u, share) + (threadIdx.x & 3), p.total[u] - 1);
            const quad_t v = *reinterpret_cast<const quad_t *>(p.t[u] + blockIdx.y * p.gs[u] + place_of(u, q));
#pragma unroll
            for (int k = 0; k < 4; ++k) none += (v[k] & 0x7fffffffu) == 0 ? 1u << 16 * u : 0;
            if (u == 0) negative = (v[0] | v[1] | v[2] | v[3]) >> 31;
            if (u == which) mine = v & 0x7fffffffu;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) sum += __uint_as_float(mine[k]);
        none = wave_sum(none);
        sum = wave_sum(sum);
        negative = __ballot(negative != 0) ? 1 : 0;
        if ((threadIdx.x & 63) == 0) {
            const int w = threadIdx.x >> 6;
            words[0][w] = none; words[1][w] = negative; words[2][w] = __float_as_uint(sum);
        }
        __syncthreads();
        none = negative = 0;
        sum = 0.f;
#pragma unroll
        for (int w = 0; w < kRangeThreads / 64; ++w) {
            none += words[0][w]; negative |= words[1][w]; sum += __uint_as_float(words[2][w]);
        }
        const unsigned left = 4 * kRangeThreads - (which ? none >> 16 : none & 0xffff);
        const unsigned mean = __float_as_uint(sum / (float)left);
        tiny_line = mean > kTinyBinades << 23 ? mean - (kTinyBinades << 23) : 0;
        fine_line = __float_as_uint(__uint_as_float(mean) * kFineShare);
        const float kept = p.dense * (1.f - (none & 0xffff) / (4.f * kRangeThreads)) * (1.f - (none >> 16) / (4.f * kRangeThreads));
        if ((p.signed_only && !negative) || split_segments(kept, false, p.steps) == 0) {
            if (blockIdx.x == 0 && threadIdx.x == 0) out->none = 1;
            return;
        }
        if (b == 0) {
            unsigned below = 0;                                  // fine ones, + 2^16 of those with few bits
#pragma unroll
            for (int k = 0; k < 4; ++k) below += mine[k] - 1u >= fine_line ? 0 : (mine[k] & 0x30000u) == 0 ? 0x10001u : 1u;
            below = wave_sum(below);
            if ((threadIdx.x & 63) == 0) words[3][threadIdx.x >> 6] = below;
            __syncthreads();
            below = 0;
#pragma unroll
            for (int w = 0; w < kRangeThreads / 64; ++w) below += words[3][w];
            if (threadIdx.x == 0) {
                out->most_big[which] = (int)(mean >> 23) + kMostAbove;
                out->few_bits[which] = 2 * (below >> 16) > (below & 0xffffu);
            }
        }
        __syncthreads();
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) out->none = 0;
    unsigned big = 0, small = 0xffffffffu, zeros = 0, signs = 0, tiny = 0, fine = 0;
    constexpr int UN = 2;
    constexpr unsigned step = kRangeBlocks * kRangeThreads;
    for (unsigned i = b * kRangeThreads + threadIdx.x; i < total; i += UN * step) {
        quad_t v[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const unsigned q = min(i + u * step, total - 1);
            v[u] = *reinterpret_cast<const quad_t *>(t + place_of(which, q));
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            unsigned none = 0, little = 0, least = 0xffffffffu;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const unsigned m = v[u][k] & 0x7fffffffu;
                signs |= v[u][k];
                big = max(big, m);
                least = min(least, m - 1u);
                none += m == 0;
                little += m - 1u < fine_line;
            }
            if (i + u * step < total) { zeros += none; fine += little; }
            small = min(small, least);
            if (__ballot(least < tiny_line) != 0) {              // seldom
#pragma unroll
                for (int k = 0; k < 4; ++k) tiny += (v[u][k] & 0x7fffffffu) - 1u < tiny_line && i + u * step < total;
            }
        }
    }
    big = wave_max(big);
    small = wave_min(small);
    zeros = wave_sum(zeros);
    tiny = wave_sum(tiny);
    fine = wave_sum(fine);
    signs = __ballot(signs >> 31) ? 1 : 0;
    if ((threadIdx.x & 63) == 0) {
        const int w = threadIdx.x >> 6;
        words[0][w] = big; words[1][w] = small; words[2][w] = zeros; words[3][w] = signs; words[4][w] = tiny; words[5][w] = fine;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < kRangeThreads / 64; ++w) {
            big = max(big, words[0][w]);
            small = min(small, words[1][w]);
            zeros += words[2][w];
            signs |= words[3][w];
            tiny += words[4][w];
            fine += words[5][w];
        }
        // (a block's tiny ones need counting up to what condemns the tensor: 2^29 operands, 2^-14 of them)
        const unsigned low = small == 0xffffffffu ? 255u : (small + 1u) >> 23;
        out->ends[which][b] = big >> 23 | (255u - low) << 8 | min(tiny, 0xffffu) << 16;
        out->zeros[which][b] = zeros | signs << 31;
        out->fine[which][b] = fine;
        if (b == 0) out->operand[which] = 0.25f / (float)total;
    }
}

// From the blocks' findings, by a wavefront whose lanes are all active (each half for one tensor), for sums of `steps` steps of 16
// products; dense: the share of these that no padding makes zero.  Latency at the head of its kernels: all loads go out together.
__device__ __forceinline__ SplitInfo split_info(const SplitRanges *r, int lane, int steps, float dense)
{
    if (uniform(r->none)) return {0, 0.f, 0.f, 0.f};
    const int t = lane >> 5, at = (lane & 31) * 2;
    const u32x4 *const ends = reinterpret_cast<const u32x4 *>(r->ends[t]) + at, *const zeros = reinterpret_cast<const u32x4 *>(r->zeros[t]) + at;
    const u32x4 *const fine = reinterpret_cast<const u32x4 *>(r->fine[t]) + at;
    unsigned big = 0, low = 0, tiny = 0, none = 0, few = 0, negative = 0;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const u32x4 e = ends[k], z = zeros[k], f = fine[k];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            big = max(big, e[i] & 0xffu);
            low = max(low, e[i] & 0xff00u);
            tiny += e[i] >> 16;
            none += z[i] & 0x7fffffffu;
            few += f[i];
            negative |= z[i];
        }
    }
    big = half_max(big);
    low = half_max(low);
    tiny = half_sum(tiny);
    none = half_sum(none);
    few = half_sum(few);
    const uint64_t signs = __ballot(negative >> 31 != 0);
    const bool one_sign = (unsigned)signs == 0 || (unsigned)(signs >> 32) == 0;
    bool fits = true;
    int e[2];
    float scale[2], kept = dense, some = 1.f, coarse = 1.f;      // products of the shares that are not zero, not fine
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const auto of = [&](unsigned v) { return (unsigned)__builtin_amdgcn_readlane((int)v, u * 32 + 31); };
        const float left = 1.f - (float)of(none) * r->operand[u];
        kept *= left;
        some *= left;
        coarse *= left - (float)of(few) * r->operand[u];
        const int top = (int)of(big);
        e[u] = top == 0 ? 0 : top - 127;
        fits = fits && e[u] >= -45 && e[u] <= 40 && 255 - (int)(of(low) >> 8) >= top - 31 &&
               top <= r->most_big[u] && (float)of(tiny) * r->operand[u] <= kMostTiny * left && !r->few_bits[u];
        scale[u] = __uint_as_float((unsigned)(127 + 14 - e[u]) << 23);
    }
    SplitInfo o;
    o.segments = fits && coarse <= (1.f - kLeastFine) * some ? split_segments(fmaxf(kept, 0.f), one_sign, steps) : 0;
    o.sa = scale[0];
    o.sb = scale[1];
    o.unscale = __uint_as_float((unsigned)(127 - 28 + e[0] + e[1]) << 23);
    return o;
}
static_assert(kRangeBlocks == 256, "eight blocks to a lane");

// two operands -> the parts of s times them, two to a word; s4096 = 4096 s.  Seven instructions, of which the last two, remainder
// and conversion in one, issue at half rate.
__device__ __forceinline__ void split_pair_two(float a, float b, float s, float s4096, unsigned &h, unsigned &l)
{
    const float a4 = a * s4096, b4 = b * s4096;
    h = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){a * s, b * s}, f16x2));
    asm("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(l) : "v"(h), "s"(-kHalfLow), "v"(a4));
    asm("v_fma_mixhi_f16 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(l) : "v"(h), "s"(-kHalfLow), "v"(b4));
}
__device__ __forceinline__ void split_eight_two(const float (&v)[8], float s, u32x4 (&o)[3])
{
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        unsigned h, l;
        split_pair_two(v[2 * t], v[2 * t + 1], s, s * kHalfLow, h, l);
        o[0][t] = h; o[1][t] = l;
    }
}

// OR of the waves' flags f in every wave; `words` is LDS that nothing else is in after the first barrier
template <int NW>
__device__ __forceinline__ int split_group_or(int *words, int wave, int lane, int f)
{
    __syncthreads();
    if (lane == 0) words[wave] = f;
    __syncthreads();
    int all = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) all |= words[i];
    return uniform(all);
}

__device__ __forceinline__ bool is_nan_bits(unsigned u) { return (u & 0x7fffffffu) > 0x7f800000u; }

// The end of every split kernel: acc becomes the sums (in: of h h'; low: of the smaller products), and the result says
// whether the work-group has to compute its tile again in fp32.  That is so where a sum to be stored is infinite; and where
// one is NaN without a NaN among the operands of its row or its column (sums that overflow to both sides, an operand from
// 2^104 on times zero).  scan(rows, columns) marks those that have one, from this wave's share of the tile's operands.
// Value v of block (i, jn) is row `row` + 32 i + 8 (v / 4) + v % 4 and column `col` + 32 jn of the tile of BM x BN; rows
// from `rows` on are not stored.  `words`: 16 + BM + BN words of LDS that nothing is in after a barrier.
template <int TM, int TN, int NW, int BM, int BN, typename Scan>
__device__ __forceinline__ bool split_finish(f32x16 (&acc)[TM][TN], const f32x16 (&low)[TM][TN], int row, int rows, int col,
                                             const bool (&col_ok)[TN], int *words, int wave, int lane, Scan scan)
{
    float probe = 0.f;                  // NaN where some sum is not finite
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int jn = 0; jn < TN; ++jn)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                acc[i][jn][v] = (acc[i][jn][v] + low[i][jn][v]) * kSplitUnscale;
                probe = fmaf(acc[i][jn][v], 0.f, probe);
            }
    bool inf = false, nan = false;
    int left = rows - row;
    asm("" : "+v"(left));              // or the compiler keeps the rows' numbers and masks in registers from here to the stores
    if (__ballot(probe != 0.f)) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int jn = 0; jn < TN; ++jn)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const unsigned s = __float_as_uint(acc[i][jn][v]);
                    const bool stored = col_ok[jn] && i * 32 + (v >> 2) * 8 + (v & 3) < left;
                    inf |= stored && (s & 0x7fffffffu) == 0x7f800000u;
                    nan |= stored && is_nan_bits(s);
                }
    }
    const int f = split_group_or<NW>(words, wave, lane, (__ballot(inf) ? 1 : 0) | (__ballot(nan) ? 2 : 0));
    if (f & 1) return true;
    if (!(f & 2)) return false;
    int *const marks = words + 16;
    for (int i = wave * 64 + lane; i < BM + BN; i += NW * 64) marks[i] = 0;
    __syncthreads();
    scan(marks, marks + BM);
    __syncthreads();
    bool open = false;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int jn = 0; jn < TN; ++jn) {
            const bool here = col_ok[jn] && !marks[BM + col + jn * 32];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int d = i * 32 + (v >> 2) * 8 + (v & 3);
                open |= here && d < left && is_nan_bits(__float_as_uint(acc[i][jn][v])) && !marks[row + d];
            }
        }
    return split_group_or<NW>(words, wave, lane, __ballot(open) ? 1 : 0) != 0;
}

// The end of a segment: the leading 8 bits of the sum of the leading products are put aside, in LDS, and what follows adds to a
// small number again.  `aside`: this thread's first 16 bytes of TM * TN * 2 rows of NW * 64, zero at first.
template <int NW, int TM, int TN>
__device__ __forceinline__ void split_clear_aside(char *aside)
{
#pragma unroll
    for (int t = 0; t < TM * TN * 2; ++t) *reinterpret_cast<u32x4 *>(aside + t * (NW * 64 * 16)) = (u32x4){0, 0, 0, 0};
}
template <int NW, int TM, int TN>
__device__ __forceinline__ void split_put_aside(f32x16 (&acc)[TM][TN], char *aside)
{
#pragma unroll
    for (int t = 0; t < TM * TN * 2; ++t) {
        f32x16 &sum = acc[t / 2 / TN][t / 2 % TN];
        u32x4 *const at = reinterpret_cast<u32x4 *>(aside + t * (NW * 64 * 16));
        u32x4 o = *at;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int v = t % 2 * 8 + 2 * k;
            const float a = sum[v] + __uint_as_float(o[k] << 16), b = sum[v + 1] + __uint_as_float(o[k] & 0xffff0000u);
            o[k] = __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2){a, b}, bf16x2));
            sum[v] = a - __uint_as_float(o[k] << 16);
            sum[v + 1] = b - __uint_as_float(o[k] & 0xffff0000u);
        }
        *at = o;
    }
}
// acc becomes the sums
template <int NW, int TM, int TN>
__device__ __forceinline__ void split_take_back(f32x16 (&acc)[TM][TN], const f32x16 (&low)[TM][TN], const char *aside, float unscale)
{
#pragma unroll
    for (int t = 0; t < TM * TN * 2; ++t) {
        f32x16 &sum = acc[t / 2 / TN][t / 2 % TN];
        const f32x16 &rest = low[t / 2 / TN][t / 2 % TN];
        const u32x4 o = *reinterpret_cast<const u32x4 *>(aside + t * (NW * 64 * 16));
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int v = t % 2 * 8 + 2 * k;
            sum[v] = (__uint_as_float(o[k] << 16) + fmaf(rest[v], kHalfLowInv, sum[v])) * unscale;
            sum[v + 1] = (__uint_as_float(o[k] & 0xffff0000u) + fmaf(rest[v + 1], kHalfLowInv, sum[v + 1])) * unscale;
        }
    }
}

// ---------------------------------------------------------------------------
// Preparation, one launch:
//   blocks [0, xb_blocks): xs[n][channel block of 16][part][Hp][Wp][16] from NCHW fp32 src (samples src_bs elements
//       apart), zeros in the padding and in channels past a column's last; one thread per (position, 8 channels), so
//       that a wavefront's stores are 1 KB runs and its loads 128-byte runs of two planes
//   the rest: wt[step = (channel block, r, s)][part][Mpad][16] from KCRS filters, the two 8-channel halves of a row
//       swapped where (row >> 3) & 1: a linear copy into LDS then lets the 16 lanes of a fragment read cover all banks;
//       one thread per 8 channels
// fold > 1 (forward of few-channel layers): the stride x stride input positions that one output position moves past become
//       channels, v = (c * fold + a) * fold + b of input row h * fold + a and column w * fold + b, so that a 3-channel 11x11
//       stride-4 layer is a 48-channel 3x3 stride-1 one: 27 steps instead of 121 of which 13 of 16 channels are zero (128 x 3 x 224 x 224, 96 filters: 296 us in fp32 with
//       the input rows in LDS -> 238 us, 37 of them this launch).
// A grouped layer's columns follow each other in both (CBg channel blocks per column, filters one column after another).
// Bound: HBM, 4 bytes read and 6 * Hp*Wp / (LH*LW) written per activation.
// ---------------------------------------------------------------------------
struct SplitPrepArgs {
    const float *src;
    u32x4 *xs;
    int64_t src_bs;
    int Cg, CBg, CBt;          // channels and channel blocks per column, channel blocks of all columns
    int LH, LW, Hp, Wp, pad_h, pad_w;
    unsigned positions;        // N * CBt * Hp * Wp
    int xb_blocks;
    const float *w;
    u32x4 *wt;
    int M, Mpad, RS, C;        // C: channels per filter (the row stride of w)
    int transposed;            // backward-data: rows are the filter's channels, reduction runs over the filters
    unsigned wt_chunks;        // groups * CBg * RS * Mpad * 2
    int64_t w_gs;              // floats between the columns' filters
    int Cin, R, S, rows, cols;               // fold > 1: input channels, the filter's and the input's extents
    int pairs;                 // fold > 1: two columns b, b + 1 are inside or outside together and 8-byte aligned
    SplitRanges *ranges;       // TWO; units of 256 threads' work
    int units, groups;
    int steps;                 // of a sum
    float dense;               // see split_info
    FastDiv div_wp, div_hp, div_cbt, div_cbg, div_mpad, div_rs, div_sv;
};

// base[i], or zero.  The load is unconditional (base must be readable): what is done with a value that is loaded under a
// condition, its scaling here, is done under that condition too, and with it the wait for each of eight loads (the preparation
// of two columns 48 -> 128 5x5 at N = 128: 68 us, 48 so).
__device__ __forceinline__ float load_or_zero(const float *base, int64_t i, bool ok)
{
    const float e = base[ok ? i : 0];
    return ok ? e : 0.f;
}

// FOLD: the stride, or 1.  TWO: in two parts where the operands' range lets it; one wavefront of a block (for each column) puts
// together what was found of it, for up to four units of 256 threads' work, a grid apart.  128 x 384 x 13 x 13 and 128 x 96 x 27 x
// 27, forward and backward-data, mean: without what was found 25.0 us, looked up for each unit 31.0, for four 29.9 (launch of its
// own: 5 more).  Consecutive units cost 5 us where three parts of 128 x 256 x 27 x 27 are written (49.5 -> 55), four a grid apart 4.
template <int FOLD, bool TWO>
__global__ __launch_bounds__(256) void split_prepare(const SplitPrepArgs p)
{
    // up to four columns from `first` on: all; or those of this block's one unit, whose 128 positions lie in no more (a column with
    // sums long enough for two parts has 47 positions of 16 channels and more)
    __shared__ SplitInfo found[4];
    unsigned first = 0;
    if constexpr (TWO) {
        const unsigned n = (unsigned)p.groups;
        if (FOLD == 1 && n > 4) {
            const bool x = (int)blockIdx.x < p.xb_blocks;
            const unsigned i = min(blockIdx.x * 128u, p.positions - 1), k = (blockIdx.x - (unsigned)p.xb_blocks) * 128u;
            const unsigned u = x ? fastdiv(fastdiv(i, p.div_wp), p.div_hp) : fastdiv(fastdiv(k, p.div_mpad), p.div_rs);
            first = fastdiv(x ? u - fastdiv(u, p.div_cbt) * (unsigned)p.CBt : u, p.div_cbg);
        }
        const unsigned c = first + (threadIdx.x >> 6);
        if (threadIdx.x >> 6 < n) {
            const SplitInfo info = split_info(p.ranges + (c < n ? c : c - n), threadIdx.x & 63, p.steps, p.dense);
            if ((threadIdx.x & 63) == 0) found[threadIdx.x >> 6] = info;
        }
        __syncthreads();
    }
    const auto found_of = [&](unsigned g) -> const SplitInfo & { return found[g >= first ? g - first : g + p.groups - first]; };
    auto piece = [&](const int unit) {
    float v[8];
    u32x4 o[3];
    // part: pieces from one part to the next (blocks lie three parts apart, also in two: columns differ)
    auto split = [&](u32x4 *dst, size_t part, unsigned g, int t, bool ok) {
        if (!ok) return;
        if (TWO && found_of(g).segments) {
            split_eight_two(v, t ? found_of(g).sb : found_of(g).sa, o);
        } else {
            split_eight(v, o);
            dst[2 * part] = o[2];
        }
        dst[0] = o[0];
        dst[part] = o[1];
    };
    if (unit < p.xb_blocks) {
        const unsigned e = (unsigned)unit * 256u + threadIdx.x;
        const unsigned i = min(e >> 1, p.positions - 1), half = e & 1;
        const unsigned t1 = fastdiv(i, p.div_wp);                    // (n*CBt + blk)*Hp + hp
        const int wp = (int)(i - t1 * (unsigned)p.Wp);
        const unsigned t2 = fastdiv(t1, p.div_hp);                    // n*CBt + blk
        const int hp = (int)(t1 - t2 * (unsigned)p.Hp);
        const unsigned n = fastdiv(t2, p.div_cbt), blk = t2 - n * (unsigned)p.CBt;
        const unsigned g = fastdiv(blk, p.div_cbg);
        const int c0 = (int)(blk - g * (unsigned)p.CBg) * 16 + (int)half * 8;     // channel inside the column
        const int h = hp - p.pad_h, w = wp - p.pad_w;
        const bool in = (unsigned)h < (unsigned)p.LH && (unsigned)w < (unsigned)p.LW;
        const int LHW = p.LH * p.LW;
        const float *const x = p.src + (int64_t)n * p.src_bs;
        if constexpr (FOLD > 1) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int ch = c0 + k, c = ch / (FOLD * FOLD), a = ch / FOLD % FOLD, b = ch % FOLD;
                const int hh = hp * FOLD + a - p.pad_h, ww = wp * FOLD + b - p.pad_w;
                const bool ok = c < p.Cin && (unsigned)hh < (unsigned)p.rows && (unsigned)ww < (unsigned)p.cols;
                const int64_t e = (int64_t)c * p.rows * p.cols + hh * p.cols + ww;
                if (FOLD % 2 == 0 && p.pairs) {
                    if (k & 1) continue;
                    const float2 t = *reinterpret_cast<const float2 *>(x + (ok ? e : 0));
                    v[k] = ok ? t.x : 0.f; v[k + 1] = ok ? t.y : 0.f;
                } else {
                    v[k] = load_or_zero(x, e, ok);
                }
            }
        } else {
            int64_t e = (int64_t)((int)g * p.Cg + c0) * LHW + h * p.LW + w;
#pragma unroll
            for (int k = 0; k < 8; ++k, e += LHW) v[k] = load_or_zero(x, e, in && c0 + k < p.Cg);
        }
        const unsigned plane = (unsigned)p.Hp * (unsigned)p.Wp;
        split(p.xs + ((size_t)t2 * 3 * plane + (i - t2 * plane)) * 2 + half, (size_t)plane * 2, g, 0, (e >> 1) < p.positions);
        return;
    }
    const unsigned all = (unsigned)(unit - p.xb_blocks) * 256u + threadIdx.x, e = min(all, p.wt_chunks - 1);
    const int half = (int)(e & 1);
    const unsigned t1 = e >> 1;                                        // ((g*CBg + cb)*RS + rs)*Mpad + m
    const unsigned t2 = fastdiv(t1, p.div_mpad);
    const int m = (int)(t1 - t2 * (unsigned)p.Mpad);
    const unsigned t3 = fastdiv(t2, p.div_rs);                         // g*CBg + cb
    const int rs = (int)(t2 - t3 * (unsigned)p.RS);
    const unsigned g = fastdiv(t3, p.div_cbg);
    const int ch0 = (int)(t3 - g * (unsigned)p.CBg) * 16 + half * 8;
    const float *w = p.w + (int64_t)g * p.w_gs;
    int64_t at = (p.transposed ? (int64_t)ch0 * p.C + m : (int64_t)m * p.C + ch0) * p.RS + rs;
    const int next = p.transposed ? p.C * p.RS : p.RS;
#pragma unroll
    for (int k = 0; k < 8; ++k, at += next) {
        const int ch = ch0 + k;
        if constexpr (FOLD > 1) {
            const int rv = (int)fastdiv((uint32_t)rs, p.div_sv), sv = rs - rv * (int)p.div_sv.d;
            const int c = ch / (FOLD * FOLD), r = rv * FOLD + ch / FOLD % FOLD, sx = sv * FOLD + ch % FOLD;
            v[k] = load_or_zero(w, ((int64_t)(m * p.Cin + c) * p.R + r) * p.S + sx, m < p.M && c < p.Cin && r < p.R && sx < p.S);
        } else {
            v[k] = load_or_zero(w, at, m < p.M && ch < p.Cg);
        }
    }
    split(p.wt + ((size_t)t2 * 3 * p.Mpad + m) * 2 + (half ^ ((m >> 3) & 1)), (size_t)p.Mpad * 2, g, 1, all < p.wt_chunks);
    if (TWO && all < p.wt_chunks && t3 == g * (unsigned)p.CBg && rs == 0 && m == 0 && half == 0) p.ranges[g].info = found_of(g);
    };
    if constexpr (TWO) {
#pragma unroll 1
        for (int unit = (int)blockIdx.x; unit < p.units; unit += (int)gridDim.x) piece(unit);
    } else {
        piece((int)blockIdx.x);
    }
}

// ---------------------------------------------------------------------------
// The contraction.  Both operands go from global memory straight into LDS (dma16, conv_bf16_dma_kernels.h); one step is
// one filter tap x 16 channels: BM filter rows and BN positions of 32 bytes in each of three parts, in an LDS buffer of
// (BM + BN) * 96 bytes, three buffers.  Eight waves, one work-group per CU (four and two where many rounds follow each
// other).  A fragment of a part serves two or three products, so a 128 x 256 tile needs 24 bytes per clock through the vector
// memory path and 62 from LDS against the 60 and ~190 they deliver: unlike the one-part bf16 kernel (48 and 96) this one is
// bound by its matrix instructions:
// 71 % of its cycles, at a clock that the power limit holds to 1.94 GHz (1.38 of the 1.77 that the pipe sustains alone on
// random operands).  384 -> 384 channels 3x3, N = 128, whole call (preparation 26 us): forward 452 -> 273 us, backward-data
// 450 -> 269; N = 2: 78 -> 33; two columns 48 -> 128 5x5, N = 128: forward 474 -> 278, backward-data 499 -> 379 (48 rows
// padded to 64).
// Two parts: half the matrix work on two thirds of the bytes.  Where the next step lies is one addition from this one's place:
// multiplied out at each step, with fields of the arguments reloaded, it was 79 scalar instructions a wave and step ahead of the
// first of 12 matrix instructions.  Kernels, three parts -> two so -> two with additions: 384 -> 384 channels 228 -> 181 -> 160
// us, backward-data of the two columns 375 -> 327 -> 250; whole layers (three passes) 851 -> 645 and 1055 -> 796 us, first layer
// (three parts) 395 -> 386.  What bounds it: power (random half-precision operands sustain 1.70 PFLOP/s against bfloat16's 1.85;
// this kernel reaches 1.1), not the loads (left out: the same time) nor the LDS reads (left out: 5 % less).  A fourth
// buffer changes nothing.
// Order inside a step: h h', h l', l h', h m' while the loads of step + 2 are issued; then every fragment of the step
// has been read, so the barrier that frees its buffer comes here; m h', m m' cover the barrier and the reads of the next
// step's h and h' (each into the registers that held this step's).
// ---------------------------------------------------------------------------
// A strided backward-data is one launch over stride x stride residue classes of (h + pad, w + pad): class (a, b) meets only the
// taps r = a, a + stride, ... and s = b, b + stride, ..., and over its own grid of positions it is a stride-1 pass over dy.
// (24 x 40 x 31 x 45, 72 filters 3x3 stride 2, whole call:
// 95 us with all taps and masks in fp32 -> 26 us.)  Forward and stride-1
// backward-data are the one-class case.
constexpr int kMaxClasses = 16;
struct SplitClass {
    int R, S;                  // taps
    int OH, OW, ncols;         // grid of positions, over all samples
    int ty, tx;                // sign -1: tap (r, s) of grid position (oh, ow) reads padded (oh + ty - r, ow + tx - s)
    int add_h, add_w;          // position (0, 0) reads src row add_h, column add_w under tap (0, 0)
    int tap0;                  // filter tap of (0, 0)
    int h0, w0;                // output row, column of grid position (0, 0)
    int first, ntiles, steps_per_split;      // first unit of the class, column tiles
    FastDiv div_plane, div_ow, div_rs, div_s;
};

struct ColGemmSplitArgs {
    const void *At;            // wt (see above)
    const void *xs;            // split, blocked, padded activations
    float *dst;                // y or dx
    float *part;               // ksplit > 1: partial outputs [ksplit][N][M][OH*OW] per column
    int M, Mpad;
    int mul;                   // input rows (columns) between grid positions
    int out_w, out_plane, out_step;          // output row and plane; rows (columns) between grid positions
    int tap_r, tap_s, RS;      // filter taps between rows, columns of a class's taps; taps of a filter
    int Wp;
    unsigned plane_bytes;      // one part of one channel block: Hp * Wp * 32
    unsigned n_blocks;         // channel blocks of all columns
    const SplitRanges *ranges; // kernels with TWO
    int N, sign;               // sign +1: tap (r, s) reads padded (oh*mul + r, ow*mul + s); -1: see SplitClass
    int cblocks;               // channel blocks per column
    int dst_bs;
    int mtiles, tiles_per_xcd, ksplit, groups, nclass, units;      // units: of one column of a grouped layer
    int64_t dst_gs, part_gs;   // floats between the columns
    // the fp32 tensors, for a tile that has to be computed in fp32
    const float *w, *src;
    int64_t w_gs, src_gs;
    int src_bs, LH, LW, Cg, C, transposed;
    int src_mul, fold, fR, fS; // rows of src between grid positions; fold and the filter's extents (see split_prepare)
    int epi_on;
    Epilogue epi;
    SplitClass cls[kMaxClasses];
};

// LDS of a work-group: three buffers of a step's operands, two parts with the sums put aside
template <int TM, int TN, int WM, int WN, bool TWO>
constexpr int split_lds()
{
    const int rows = (TM * WM + TN * WN) * 32, three = 3 * rows * 96, two = 3 * rows * 64 + TM * TN * WM * WN * 64 * 32;
    return TWO && two > three ? two : three;
}

template <int TM, int TN, int WM, int WN, bool TWO>
__global__ __launch_bounds__(WM * WN * 64, WM * WN == 4 ? 2 : 1) void colgemm_split_kernel(const ColGemmSplitArgs p)
{
    constexpr int NW = WM * WN;
    constexpr int BM = TM * WM * 32, BN = TN * WN * 32;
    constexpr int MPG = TM * TN;                               // matrix instructions per product
    static_assert(NW == 8 || NW == 4, "eight waves, or four and two work-groups per CU");
    static_assert(split_lds<TM, TN, WM, WN, TWO>() * (8 / NW) <= 160 * 1024, "LDS buffers");

    extern __shared__ __attribute__((aligned(16))) float lds_fast[];
    const char *const lds = reinterpret_cast<const char *>(lds_fast);
    const unsigned lds_base = (unsigned)(size_t)lds_fast;

    const int bid = blockIdx.x;
    const int idx = bid >> 3;
    const int unit = (bid & 7) * p.tiles_per_xcd + idx;
    if (idx >= p.tiles_per_xcd || unit >= p.units * p.groups) return;
    const int gcol = unit / p.units;
    int unit_c = unit - gcol * p.units;
    int ci = 0;
    while (ci + 1 < p.nclass && unit_c >= p.cls[ci + 1].first) ++ci;
    const SplitClass &q = p.cls[ci];
    unit_c -= q.first;
    const int ntile = p.mtiles * q.ntiles;
    const int ks = unit_c / ntile;
    const int tile = unit_c - ks * ntile;
    const int mt = tile % p.mtiles, nt = tile / p.mtiles;
    const int m0 = mt * BM, n0 = nt * BN;

    SplitInfo info = {0, 0.f, 0.f, 0.f};
    if constexpr (TWO) {
        info.segments = uniform(p.ranges[gcol].info.segments);
        info.unscale = __int_as_float(uniform(__float_as_int(p.ranges[gcol].info.unscale)));
    }
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = uniform(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;

    const int step_begin = ks * q.steps_per_split;
    const int nsteps = max(0, min(p.cblocks * q.R * q.S - step_begin, q.steps_per_split));
    f32x16 acc[TM][TN], low[TM][TN];           // sums of h h'; of the five smaller products
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int jn = 0; jn < TN; ++jn)
#pragma unroll
            for (int v = 0; v < 16; ++v) { acc[i][jn][v] = 0.f; low[i][jn][v] = 0.f; }

    const int l32 = lane & 31, half = lane >> 5;

    auto contract = [&](auto parts_c) {
    constexpr unsigned PARTS = decltype(parts_c)::value;
    constexpr int QA = BM * PARTS / 32, QB = BN * PARTS / 32;  // 1 KB loads per step: filters, activations
    constexpr int NL = (QA + QB + NW - 1) / NW;                // ... per wave (the last may repeat an earlier one)
    constexpr int BUF = (BM + BN) * PARTS * 32;

    // Load i of this wave is 1 KB block q of the step: 32 rows of one part, filters first.  LDS block q lies at q * 1024.
    unsigned voff[NL], lq[NL];
    bool isa[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        int lb = i * NW + wave;
        if ((i + 1) * NW > QA + QB && lb >= QA + QB) lb -= NW;   // repeats this wave's previous load
        lq[i] = (unsigned)lb * 1024u;
        isa[i] = (i + 1) * NW <= QA || (i * NW < QA && lb < QA);
        if (isa[i]) {
            const int c = lb / (BM / 32), b = lb - c * (BM / 32);
            voff[i] = (unsigned)((c * p.Mpad + b * 32) * 32 + lane * 16);
        } else {
            const int qb = lb - QA;
            const int c = qb / (BN / 32), b = qb - c * (BN / 32);
            const int row = b * 32 + (lane >> 1);
            const int chunk = (lane & 1) ^ ((row >> 3) & 1);
            int j = n0 + row;
            j = j < q.ncols ? j : 0;                             // columns past the end: computed, never stored
            const int n = (int)fastdiv((uint32_t)j, q.div_plane);
            const int rem = j - n * (q.OH * q.OW);
            const int oh = (int)fastdiv((uint32_t)rem, q.div_ow);
            const int ow = rem - oh * q.OW;
            voff[i] = (unsigned)n * p.n_blocks * (3 * p.plane_bytes) + (unsigned)c * p.plane_bytes +
                      (unsigned)((oh * p.mul * p.Wp + ow * p.mul) * 32 + chunk * 16);
        }
    }

    // Where the next step to load lies, and how far it is to the one after: the next column of taps, the next row, the next
    // channel block (one addition each: a wave issues one scalar instruction in four clocks and has few clocks a step).
    const int CR = q.R, CS = q.S;
    const int a_step_bytes = p.Mpad * 96;
    const int64_t cb_bytes = (int64_t)3 * p.plane_bytes;
    const char *a_base = nullptr, *xs = nullptr;
    int left_r = 0, left_s = 0;                                  // rows and columns of taps from here on
    auto seek = [&](int st) {
        const int cb = (int)fastdiv((uint32_t)st, q.div_rs);
        const int rs = st - cb * (CR * CS);
        const int r = (int)fastdiv((uint32_t)rs, q.div_s), s = rs - r * CS;
        a_base = static_cast<const char *>(p.At) + (size_t)m0 * 32 +
                 ((int64_t)(gcol * p.cblocks + cb) * p.RS + q.tap0 + r * p.tap_r + s * p.tap_s) * a_step_bytes;
        const int ar = p.sign > 0 ? r : q.ty - r, as = p.sign > 0 ? s : q.tx - s;
        xs = static_cast<const char *>(p.xs) + (gcol * p.cblocks + cb) * cb_bytes + (ar * p.Wp + as) * 32;
        left_r = CR - r; left_s = CS - s;
    };
    const int a_s = p.tap_s * a_step_bytes, a_r = (p.tap_r - (CS - 1) * p.tap_s) * a_step_bytes;
    const int a_c = (p.RS - (CR - 1) * p.tap_r - (CS - 1) * p.tap_s) * a_step_bytes;
    const SplitSteps x_step = split_steps(p.plane_bytes, p.Wp, CR, CS, p.sign);
    auto advance = [&]() {
        int da = a_s;
        int64_t dx = x_step.s;
        left_s -= 1;
        if (left_s == 0) {
            left_s = CS; da = a_r; dx = x_step.r;
            left_r -= 1;
            if (left_r == 0) { left_r = CR; da = a_c; dx = x_step.c; }
        }
        a_base += da; xs += dx;
    };
    auto load_one = [&](int i, unsigned lbuf) { dma16(isa[i] ? a_base : xs, voff[i], lbuf + lq[i]); };
    auto load_step = [&](int buf) {
#pragma unroll
        for (int i = 0; i < NL; ++i) load_one(i, lds_base + buf * BUF);
        advance();
    };

    const int choff = (half ^ ((l32 >> 3) & 1)) * 16;
    const int a_row = (wm * TM * 32 + l32) * 32 + choff;
    const int b_row = BM * PARTS * 32 + (wn * TN * 32 + l32) * 32 + choff;
    auto read_a = [&](int bufo, int c, u32x4 (&f)[TM]) {
#pragma unroll
        for (int i = 0; i < TM; ++i) f[i] = *reinterpret_cast<const u32x4 *>(lds + bufo + a_row + (c * BM + i * 32) * 32);
    };
    auto read_b = [&](int bufo, int c, u32x4 (&f)[TN]) {
#pragma unroll
        for (int jn = 0; jn < TN; ++jn) f[jn] = *reinterpret_cast<const u32x4 *>(lds + bufo + b_row + (c * BN + jn * 32) * 32);
    };

    seek(step_begin);
    if (nsteps > 0) load_step(0);
    if (nsteps > 1) load_step(1);
    if (nsteps > 1) wait_vmcnt<NL>(); else wait_vmcnt<0>();
    __syncthreads();
    int step = 0, bufo = 0;                                      // this step's buffer, in bytes
    const auto after = [&](int o) { return o == 2 * BUF ? 0 : o + BUF; };

    if constexpr (PARTS == 2) {
        // Order inside a step: h h' and h l' while the loads of step + 2 are issued; the barrier, behind which the next step's
        // h and h' are read into a second set of registers; l h'.
        constexpr int SLOTS = 2 * MPG, SPACING = SLOTS / NL > 0 ? SLOTS / NL : 1;
        u32x4 ha[2][TM], hb[2][TN], la[TM], lb[TN];
        if (nsteps > 0) { read_a(0, 0, ha[0]); read_b(0, 0, hb[0]); }
        // (the last steps load the last one again: one form of the step, or the sums change registers between its forms)
        int to_load = nsteps - 2;
        if (to_load <= 0) seek(step_begin + nsteps - 1);
        auto do_step = [&](auto set_c) {
            constexpr int set = decltype(set_c)::value;
            const int bufo1 = after(bufo);
            const unsigned lbuf = lds_base + after(bufo1);
            auto product = [&](const u32x4 (&xa)[TM], const u32x4 (&xb)[TN], auto g_c) {
                constexpr int g = decltype(g_c)::value;
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int jn = 0; jn < TN; ++jn) {
                        f32x16 &sum = g == 0 ? acc[i][jn] : low[i][jn];
                        sum = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, xa[i]),
                                                                     __builtin_bit_cast(f16x8, xb[jn]), sum, 0, 0, 0);
                        const int m = g * MPG + i * TN + jn;
                        if (g < 2) {
#pragma unroll
                            for (int u = 0; u < NL; ++u)
                                if ((u * SPACING < SLOTS ? u * SPACING : SLOTS - 1) == m) {
                                    __builtin_amdgcn_sched_barrier(0);
                                    load_one(u, lbuf);
                                    __builtin_amdgcn_sched_barrier(0);
                                }
                        }
                    }
                __builtin_amdgcn_sched_barrier(0);
            };
            read_b(bufo, 1, lb);
            read_a(bufo, 1, la);
            __builtin_amdgcn_sched_barrier(0);
            product(ha[set], hb[set], I<0>{});
            product(ha[set], lb, I<1>{});
            to_load -= 1;
            if (to_load > 0) advance();
            wait_vmcnt<NL>();
            asm volatile("s_waitcnt lgkmcnt(0)");
            __syncthreads();
            read_a(bufo1, 0, ha[set ^ 1]);
            read_b(bufo1, 0, hb[set ^ 1]);
            __builtin_amdgcn_sched_barrier(0);
            product(la, hb[set], I<2>{});
            ++step;
            bufo = bufo1;
        };
        char *const aside = const_cast<char *>(lds) + 3 * BUF + tid * 16;
        split_clear_aside<NW, TM, TN>(aside);
        const int segment = nsteps / info.segments;
        int segment_end = segment;
        while (step + 1 < nsteps) {
            if (step >= segment_end) {
                split_put_aside<NW>(acc, aside);
                segment_end += segment;
            }
            do_step(I<0>{});
            do_step(I<1>{});
        }
        if (step < nsteps) do_step(I<0>{});
        wait_vmcnt<0>();
        split_take_back<NW>(acc, low, aside, info.unscale);
    } else {
    constexpr int SLOTS = 4 * MPG;                              // matrix instructions before the barrier
    constexpr int SPACING = SLOTS / NL > 0 ? SLOTS / NL : 1;
    u32x4 fa[3][TM], fb[3][TN];                                // fragments, by part
    if (nsteps > 0) { read_a(0, 0, fa[0]); read_b(0, 0, fb[0]); }
    auto do_step = [&](auto more_c) {                           // more: the loads of step + 2 exist
        constexpr bool more = decltype(more_c)::value;
        const int bufo1 = after(bufo);
        const unsigned lbuf = lds_base + after(bufo1);
        const bool next = more || step + 1 < nsteps;
        // product g of this step: part ca of the filters with part cb of the activations
        auto product = [&](int ca, int cb, int g) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int jn = 0; jn < TN; ++jn) {
                    f32x16 &sum = g == 0 ? acc[i][jn] : low[i][jn];
                    sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fa[ca][i]),
                                                                  __builtin_bit_cast(bf16x8, fb[cb][jn]), sum, 0, 0, 0);
                    const int m = g * MPG + i * TN + jn;
                    if (more && g < 4) {
#pragma unroll
                        for (int u = 0; u < NL; ++u)
                            if ((u * SPACING < SLOTS ? u * SPACING : SLOTS - 1) == m) {
                                __builtin_amdgcn_sched_barrier(0);
                                load_one(u, lbuf);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                    }
                }
            __builtin_amdgcn_sched_barrier(0);
        };
        read_b(bufo, 2, fb[2]);
        read_a(bufo, 2, fa[2]);
        __builtin_amdgcn_sched_barrier(0);
        product(0, 0, 0);
        read_b(bufo, 1, fb[1]);
        read_a(bufo, 1, fa[1]);
        __builtin_amdgcn_sched_barrier(0);
        product(0, 2, 1);
        product(2, 0, 2);
        product(0, 1, 3);
        if (more) advance();
        if (more) wait_vmcnt<NL>(); else wait_vmcnt<0>();
        asm volatile("s_waitcnt lgkmcnt(0)");
        __syncthreads();
        if (next) read_a(bufo1, 0, fa[0]);
        __builtin_amdgcn_sched_barrier(0);
        product(1, 0, 4);
        if (next) read_b(bufo1, 0, fb[0]);
        __builtin_amdgcn_sched_barrier(0);
        product(1, 1, 5);
        ++step;
        bufo = bufo1;
    };
    while (step + 2 < nsteps) do_step(std::true_type{});
    while (step < nsteps) do_step(std::false_type{});

    // sums that call for fp32 arithmetic: the whole work-group computes its tile again
    {
        bool col_ok[TN];
#pragma unroll
        for (int jn = 0; jn < TN; ++jn) col_ok[jn] = n0 + (wn * TN + jn) * 32 + l32 < q.ncols;
        auto scan = [&](int *nan_rows, int *nan_cols) {
            // A filter padded to whole strides has zeros over real input: there a NaN input makes a sum NaN that its window
            // does not call for.
            const bool padded = p.fold > 1 && (p.fR % p.fold != 0 || p.fS % p.fold != 0);
#pragma unroll 1
            for (int st = step_begin; st < step_begin + nsteps; ++st) {
                seek(st);
#pragma unroll
                for (int i = 0; i < NL; ++i) {                   // the blocks of h parts: rows b * 32 + lane / 2
                    const int lb = (int)(lq[i] / 1024u), b = isa[i] ? lb : lb - QA;
                    if (isa[i] ? b >= BM / 32 : b >= BN / 32 || padded) continue;
                    const u32x4 e = *reinterpret_cast<const u32x4 *>((isa[i] ? a_base : xs) + voff[i]);
                    bool nan = false;
#pragma unroll
                    for (int t = 0; t < 4; ++t) nan |= is_nan_bits(e[t] & 0xffff0000u) || is_nan_bits(e[t] << 16);
                    if (nan) (isa[i] ? nan_rows : nan_cols)[b * 32 + (lane >> 1)] = 1;
                }
            }
        };
        if (split_finish<TM, TN, NW, BM, BN>(acc, low, wm * TM * 32 + half * 4, p.M - m0, wn * TN * 32 + l32, col_ok,
                                             reinterpret_cast<int *>(lds_fast), wave, lane, scan)) {
            const float *const wg = p.w + (size_t)gcol * p.w_gs;
            const float *const sg = p.src + (size_t)gcol * p.src_gs;
            int rowm[TM], hb[TN], wb[TN];
            int64_t base[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) rowm[i] = m0 + (wm * TM + i) * 32 + l32;
#pragma unroll
            for (int jn = 0; jn < TN; ++jn) {
                int j = n0 + (wn * TN + jn) * 32 + l32;
                j = j < q.ncols ? j : 0;
                const int n = (int)fastdiv((uint32_t)j, q.div_plane);
                const int rem = j - n * (q.OH * q.OW);
                const int oh = (int)fastdiv((uint32_t)rem, q.div_ow);
                hb[jn] = oh * p.src_mul + q.add_h;
                wb[jn] = (rem - oh * q.OW) * p.src_mul + q.add_w;
                base[jn] = (int64_t)n * p.src_bs;
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int jn = 0; jn < TN; ++jn)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[i][jn][v] = 0.f;
#pragma unroll 1
            for (int st = step_begin; st < step_begin + nsteps; ++st) {
                const int cbk = (int)fastdiv((uint32_t)st, q.div_rs);
                const int rs = st - cbk * (q.R * q.S);
                const int rr = (int)fastdiv((uint32_t)rs, q.div_s), ss = rs - rr * q.S;
                const int tap = q.tap0 + rr * p.tap_r + ss * p.tap_s;
#pragma unroll 1
                for (int t0 = 0; t0 < 8; t0 += 4) {              // the loads of four elements in flight, unconditional
                    float a[4][TM], b[4][TN];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        int ch = cbk * 16 + half * 8 + t0 + t, dh = p.sign * rr, dw = p.sign * ss, tap_e = tap;
                        bool real = true;                        // a tap of the filter (folded filters are padded)
                        if (p.fold > 1) {
                            const int ab = ch % (p.fold * p.fold);
                            ch /= p.fold * p.fold;
                            dh = rr * p.fold + ab / p.fold; dw = ss * p.fold + ab % p.fold;
                            real = dh < p.fR && dw < p.fS;
                            tap_e = dh * p.fS + dw;
                        }
                        const int taps = p.fold > 1 ? p.fR * p.fS : p.RS;
#pragma unroll
                        for (int i = 0; i < TM; ++i) {
                            const bool ok = real && rowm[i] < p.M && ch < p.Cg;
                            const int64_t o = p.transposed ? ((int64_t)ch * p.C + rowm[i]) * taps + tap_e
                                                           : ((int64_t)rowm[i] * p.C + ch) * taps + tap_e;
                            const float e = wg[ok ? o : 0];
                            a[t][i] = ok ? e : 0.f;
                        }
#pragma unroll
                        for (int jn = 0; jn < TN; ++jn) {
                            const int h = hb[jn] + dh, w = wb[jn] + dw;
                            const bool ok = real && ch < p.Cg && (unsigned)h < (unsigned)p.LH && (unsigned)w < (unsigned)p.LW;
                            const float e = sg[ok ? base[jn] + (int64_t)ch * (p.LH * p.LW) + h * p.LW + w : 0];
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

    }
    };
    if constexpr (TWO) {
        if (info.segments) contract(std::integral_constant<unsigned, 2>{});
        else contract(std::integral_constant<unsigned, 3>{});
    } else {
        contract(std::integral_constant<unsigned, 3>{});
    }

    float *const dst_c = p.dst + (size_t)gcol * p.dst_gs;
    float *const part_c = p.part + (size_t)gcol * p.part_gs;
    const int plane = p.out_plane;
#pragma unroll
    for (int jn = 0; jn < TN; ++jn) {
        const int col = n0 + (wn * TN + jn) * 32 + l32;
        if (col >= q.ncols) continue;
        const int n = (int)fastdiv((uint32_t)col, q.div_plane);
        int rem = col - n * (q.OH * q.OW);
        if (p.out_step > 1) {
            const int oh = (int)fastdiv((uint32_t)rem, q.div_ow);
            rem = (oh * p.out_step + q.h0) * p.out_w + (rem - oh * q.OW) * p.out_step + q.w0;
        }
        float *out = p.ksplit > 1 ? part_c + ((size_t)ks * p.N + n) * ((size_t)p.M * plane) + rem
                                  : dst_c + (size_t)n * p.dst_bs + rem;
        if (p.epi_on && p.ksplit == 1)            // one column only; split sums get it in reduce_split_outputs
            epi_tile<TM, TN>(p.epi, acc, jn, m0 + wm * TM * 32 + half * 4, p.M, plane,
                             (int64_t)n * p.epi.mask_bs + rem);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int row0 = m0 + (wm * TM + i) * 32 + half * 4;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = row0 + (v >> 2) * 8 + (v & 3);
                if (row < p.M) out[(size_t)row * plane] = acc[i][jn][v];
            }
        }
    }
}
