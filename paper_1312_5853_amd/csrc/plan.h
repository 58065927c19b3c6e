// Host-side planning for the convolution passes: argument checks, derived
// extents, tile-shape choice, split count of the backward-filter reduction and
// the workspace layout.  Plain C++ with no HIP dependency, so the same header
// compiles into a CPU-only self-test.
#ifndef CONVNET_PLAN_H
#define CONVNET_PLAN_H

#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <algorithm>

#include "fastdiv.h"

namespace convnet {

constexpr int kStatusOk = 0;
constexpr int kErrInvalidArg = -1;
constexpr int kErrTooLarge = -2;
constexpr int kErrBadDtype = -3;
constexpr int kErrWorkspace = -4;
constexpr int kErrMisaligned = -5;
constexpr int kErrHip = -6;
constexpr int kErrScratchLimit = -7;

constexpr int kOpFwd = 0, kOpBwdData = 1, kOpBwdFilter = 2;
constexpr int kDtypeF32 = 0, kDtypeBf16 = 1, kDtypeBf16OutBf16 = 2;

constexpr int kChunk = 16;            // reduction elements staged in LDS per step
constexpr int kTapTablePad = 256;     // tap table length is rounded up to this
constexpr int64_t kMaxSpanBytes = (int64_t)1 << 31;
constexpr int kTargetGroups = 512;    // work-groups wanted in flight: 2 per CU on 256 CUs

struct Problem {
    int N, C, H, W, K, R, S, stride, pad;
    int P, Q;
    int64_t x_bs, y_bs;               // batch strides in elements
    int dtype;                        // of the inputs: kDtypeF32 or kDtypeBf16
    bool out_bf16;                    // forward / backward-data write bf16 (caller passed kDtypeBf16OutBf16)
    // Grouped (multi-column) layer: C and K above are the PER-COLUMN counts, the batch strides those of the
    // full tensors; column g starts g * x_gs / y_gs / w_gs elements into x / y / the filters.
    int groups;
    int64_t x_gs, y_gs, w_gs;
};

// Tile shape of one work-group (4 waves): each wave owns TM x TN MFMA tiles of
// 32 x 32; waves are laid out WM x WN.
struct TileShape {
    int TM, TN, WM, WN;
    int mfma;                          // edge of the square matrix-instruction block: 32, or 16 for the 48-row tile
    int bm() const { return TM * WM * mfma; }
    int bn() const { return TN * WN * mfma; }
};

constexpr TileShape kTile128x128 = {2, 2, 2, 2, 32};
constexpr TileShape kTile96x128 = {3, 1, 1, 4, 32};
constexpr TileShape kTile64x128 = {2, 1, 1, 4, 32};
constexpr TileShape kTile32x256 = {1, 2, 1, 4, 32};
constexpr TileShape kTile48x256 = {3, 4, 1, 4, 16};   // fp32 forward / backward-data fast path only
constexpr TileShape kTile128x256 = {2, 4, 2, 2, 32};  // bf16 direct-to-LDS kernel only

inline int round_up(int v, int m) { return (v + m - 1) / m * m; }
inline int64_t round_up64(int64_t v, int64_t m) { return (v + m - 1) / m * m; }
inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Row-tile choice: the block height that pads M (rows of the GEMM view) least;
// ties go to the taller block (more reuse of the gathered operand).
inline TileShape pick_tile(int M)
{
    const TileShape cand[4] = {kTile128x128, kTile96x128, kTile64x128, kTile32x256};
    TileShape best = cand[0];
    int best_cost = round_up(M, best.bm());
    for (int i = 1; i < 4; ++i) {
        int cost = round_up(M, cand[i].bm());
        if (cost < best_cost) { best = cand[i]; best_cost = cost; }
    }
    return best;
}

inline int out_extent(int in, int filt, int stride, int pad)
{
    int span = in + 2 * pad - filt;
    return span < 0 ? 0 : span / stride + 1;
}

// Fills P, Q and checks everything that can be checked without touching the GPU.
inline int make_problem(Problem &pb, int N, int C, int H, int W, int K, int R, int S,
                        int stride, int pad, int64_t x_bs, int64_t y_bs, int dtype)
{
    if (N <= 0 || C <= 0 || H <= 0 || W <= 0 || K <= 0 || R <= 0 || S <= 0) return kErrInvalidArg;
    if (stride <= 0 || pad < 0) return kErrInvalidArg;
    if (dtype != kDtypeF32 && dtype != kDtypeBf16 && dtype != kDtypeBf16OutBf16) return kErrBadDtype;
    pb.out_bf16 = dtype == kDtypeBf16OutBf16;
    if (pb.out_bf16) dtype = kDtypeBf16;
    // keep every intermediate below 2^31 before multiplying extents together
    if (pad > (1 << 20) || stride > (1 << 20)) return kErrTooLarge;
    if ((int64_t)H + 2 * (int64_t)pad < R || (int64_t)W + 2 * (int64_t)pad < S) return kErrInvalidArg;
    pb.N = N; pb.C = C; pb.H = H; pb.W = W; pb.K = K; pb.R = R; pb.S = S;
    pb.stride = stride; pb.pad = pad; pb.dtype = dtype;
    pb.groups = 1; pb.x_gs = 0; pb.y_gs = 0; pb.w_gs = 0;
    pb.P = out_extent(H, R, stride, pad);
    pb.Q = out_extent(W, S, stride, pad);
    if (pb.P <= 0 || pb.Q <= 0) return kErrInvalidArg;
    const int64_t x_sample = (int64_t)C * H * W, y_sample = (int64_t)K * pb.P * pb.Q;
    const int64_t w_elems = (int64_t)K * C * R * S;
    if (x_bs == 0) x_bs = x_sample;
    if (y_bs == 0) y_bs = y_sample;
    if (x_bs < x_sample || y_bs < y_sample) return kErrInvalidArg;
    pb.x_bs = x_bs; pb.y_bs = y_bs;
    const int64_t fat = 4;   // widest element the kernels index with 32-bit offsets
    if (x_sample >= kMaxSpanBytes / fat || y_sample >= kMaxSpanBytes / fat) return kErrTooLarge;
    if (x_bs >= kMaxSpanBytes / fat || y_bs >= kMaxSpanBytes / fat) return kErrTooLarge;
    if ((int64_t)N * x_bs * fat >= kMaxSpanBytes) return kErrTooLarge;
    if ((int64_t)N * y_bs * fat >= kMaxSpanBytes) return kErrTooLarge;
    if (w_elems * fat >= kMaxSpanBytes) return kErrTooLarge;
    if ((int64_t)C * R * S >= (1 << 28) || (int64_t)K * R * S >= (1 << 28)) return kErrTooLarge;
    return kStatusOk;
}

// What one pass needs in the workspace, in bytes from its 256-aligned base.
struct Plan {
    int op;
    TileShape tile;
    int M;            // rows of the GEMM view: K (fwd, wgrad) or C (dgrad)
    int Mpad;
    int Kg;           // fwd: C*R*S, dgrad: K*R*S, wgrad: C*R*S (columns of dw)
    int Kgpad;        // Kg rounded up to kChunk
    int tab_len;      // tap table entries
    int kc;           // reduction depth of one step (16, or 32 where the fast path allows)
    int nsplit;       // wgrad: partial sums over the (n, p, q) reduction
    int chunks_per_split;
    size_t tab_off, tab_bytes;
    size_t wt_off, wt_bytes;          // re-laid-out filters (fwd, dgrad)
    size_t part_off, part_bytes;      // wgrad partials
    bool widen;                       // bf16 activation-side inputs are widened to dense fp32 copies first
    bool widen_w;                     // bf16 filters are widened to fp32 first (forward, backward-data)
    // forward with few channels: the input rows of a 128-position tile are staged once in LDS (patch kernel),
    // row tile of patch_tm * 32 filters, patch_nr rows of pitch patch_wp per channel, patch_lds bytes of LDS
    bool patch;
    int patch_tm, patch_nr, patch_wp, patch_lds;
    size_t cvt_off[2], cvt_bytes[2];  // bf16 -> fp32 staging of the two inputs
    size_t blk_off, blk_bytes;        // channel-blocked copy of the gathered bf16 tensor (forward, backward-data)
    size_t stage_off, stage_bytes;    // dense fp32 result of forward / backward-data before it is rounded to bf16
    // bf16 backward-filter of a stride-1 layer whose output has the input's extent: packed copies in which a
    // filter tap is a linear shift (row pitch lin_wq, lin_jy / lin_jx elements per image), 64 positions per step
    bool lin;
    int lin_wq, lin_jy, lin_jx, lin_steps;      // (a grouped layer: fused_groups, both regions hold all columns)
    size_t lin_dy_off, lin_dy_bytes, lin_x_off, lin_x_bytes;
    // columns of a grouped layer run in ONE launch (fp32 kernels of the fast paths): the filter and partial-sum
    // regions then hold `groups` consecutive copies; otherwise the host runs the columns one after the other
    bool fused_groups;
    // bf16 forward / stride-1 backward-data on the direct-to-LDS kernel: channel-blocked, zero-padded copy of the
    // gathered tensor (dma_hp x dma_wp positions per plane, dma_ph rows / dma_pw columns of zeros before the data),
    // dma_kc channels per step, dma_occ work-groups per CU
    bool dma;
    int dma_kc, dma_occ, dma_hp, dma_wp, dma_ph, dma_pw;
    size_t xb_off, xb_bytes;
    // bf16 backward-filter of a stride-4, pad-2 layer with at most four input channels on the bf16 matrix
    // instruction (input rows staged as shifted copies in LDS): rows_splits output-row ranges per image,
    // rows_wgs work-groups with one partial result each, rows_lds bytes of LDS
    bool rows;
    int rows_splits, rows_wgs, rows_lds;
    // the same decomposition for fp32 tensors (any stride up to 4): rows_wp = LDS pitch of a staged input row
    bool rows_f32;
    int rows_wp;
    bool rows_split;     // ... on three bfloat16 parts (stride 4): rows_lds is then its
    // fp32 forward / stride-1 backward-data on the bf16 matrix instruction, operands split into three bfloat16 parts
    // (colgemm_split_kernel): tile sp_bm x sp_bn, sp_cb blocks of 16 channels per column, zero-padded planes of
    // sp_hp x sp_wp positions with sp_ph / sp_pw rows / columns of zeros before the data.  The workspace then holds
    // only the regions below (nsplit, chunks_per_split as above).
    bool sp;
    // sp_fold > 1: the stride x stride input positions under an output position are channels (forward of few channels)
    // sp_pair: four-wave work-groups, two to a CU
    bool sp_pair;
    // sp_two: in two half-precision parts where the operands' range lets it; what was found of it lies at sp_range_off
    bool sp_two;
    int sp_two_steps;          // of the shortest sum (forward, backward-data)
    float sp_dense;            // share of the products that no padding makes zero
    size_t sp_range_off, sp_range_bytes;
    int sp_bm, sp_bn, sp_cb, sp_hp, sp_wp, sp_ph, sp_pw, sp_mpad, sp_fold;
    size_t sp_w_off, sp_w_bytes, sp_x_off, sp_x_bytes;
    // bf16 stride-1 forward / backward-data with the input window of a tile in LDS (colgemm_bf16_window_kernel): 64 or 128 rows,
    // win_tn blocks of 32 positions per wave, win_ncb channel blocks per step of win_cb (padded) in a column, planes of
    // win_hp x win_wp positions, win_bytes of LDS per block's window, win_lds in all
    bool win;
    int win_bm, win_tn, win_ncb, win_cb, win_hp, win_wp, win_ph, win_pw, win_bytes, win_lds;
    bool direct;                      // small problem: one launch on the vector units, no workspace read or written
    size_t total;
};

constexpr TileShape kTile128x192 = {2, 3, 2, 2, 32};  // bf16 direct-to-LDS kernel only

// Tile width, step depth and work-groups per CU of the direct-to-LDS bf16 kernel (128 rows per tile).  Width: the
// one that needs the least time on 256 CUs, rounds of tiles x columns per tile (a wider tile moves less through the
// memory path per matrix instruction, so ties go to it).  One round: 64-channel steps, one work-group per CU (three
// LDS buffers of up to 48 KB).  More rounds: 32-channel steps so that two work-groups share a CU and hide each
// other's barriers and epilogues.
inline void pick_dma_tile(int channels, int mtiles, int64_t ncols, TileShape &tile, int &kc, int &occ)
{
    const TileShape cand[3] = {kTile128x256, kTile128x192, kTile128x128};
    int64_t best = -1, best_rounds = 1;
    for (int i = 0; i < 3; ++i) {
        const int64_t tiles = mtiles * ((ncols + cand[i].bn() - 1) / cand[i].bn());
        const int64_t rounds = (tiles + 255) / 256;
        const int64_t cost = rounds * cand[i].bn();
        if (best < 0 || cost < best) { best = cost; tile = cand[i]; best_rounds = rounds; }
    }
    if (best_rounds > 1 || channels % 64 != 0) { kc = 32; occ = 2; }
    else { kc = 64; occ = 1; }
}

// One axis of a residue class of a strided backward-data: input positions h with (h + pad) % stride == cls meet the taps
// r = cls, cls + stride, ... only; h = stride * a + cls - pad reads dy at a - (r - cls) / stride.  Forward: the one class of
// all output positions.
struct ClassGrid {
    int taps, count;           // taps of the class; positions a = first, first + 1, ...
    int first, out0;           // dy (input) position of the first under the class's first tap; its output position
};
inline ClassGrid class_grid(bool fwd, int out, int taps, int stride, int pad, int cls)
{
    if (fwd) return {taps, out, -pad, 0};
    ClassGrid g;
    g.taps = taps > cls ? (taps - cls + stride - 1) / stride : 0;
    g.first = pad > cls ? (pad - cls + stride - 1) / stride : 0;
    g.out0 = stride * g.first + cls - pad;
    g.count = g.out0 < out ? (out - 1 - g.out0) / stride + 1 : 0;
    return g;
}

// Rows of a tile: what pads `rows` least, ties to the taller tile
inline int least_padding(int rows)
{
    int bm = 128;
    for (int b : {96, 64, 32})
        if (round_up(rows, b) < round_up(rows, bm)) bm = b;
    return bm;
}

// Segments: a product of two halves has 22 significant bits, so every instruction rounds the sum of the leading products; those of
// bfloat16 have 16, and leave many of their sums exact, the more the more operands are zero.  In 1e-14, squares of 2-norm errors
// against 64 bits (fitted to 170 layers, with the output of a ReLU or of pooling for input, with gradients that such layers leave
// zeros in): three parts 0.061 steps k - 0.2, k the share of products without a zero to the power of 3/4 and at most 0.7 for
// a tensor of one sign; two parts 0.058 (steps / segments + segments) + 0.95.  As few segments as make the second at most 0.92 of
// the first, each of at least 16 steps (the end of a segment costs as much as two to four steps), or three parts.
// kept: the share of products without a zero among their operands; steps: of 16 products a sum.
CONVNET_HD int split_segments(float kept, bool one_sign, int steps)
{
    kept = __builtin_sqrtf(kept * __builtin_sqrtf(kept));
    if (one_sign && kept > 0.7f) kept = 0.7f;
    const float n = (float)steps, three = 0.92f * (0.061f * n * kept - 0.2f);
    int segments = 0;
    for (int g = 8; g >= 2; g /= 2)
        if (steps >= 16 * g && 0.058f * (n / (float)g + (float)g) + 0.95f <= three) segments = g;
    return segments;
}

// Two half-precision parts instead of three bfloat16 ones (conv_split_kernels.h) where the operands let it: a pass asks for that
// where split_segments finds that dense operands would do, and where `share` of the contraction's estimated three-part time is
// more than the launch that looks at the operands costs (4.5 us and their bytes; 128 x 384 x 13 x 13 with 384 filters 3x3: 10.8 us).
// On 170 drawn passes of enough steps two parts took, of three parts' time: forward 0.71 and backward-data 0.65 (each of 104 less;
// under the line, which the smallest calls are, up to 0.98), backward-filter 0.77 (0.95 and less above the line, up to 1.10 under
// it: its share is the smaller one, the operands of its short sums being the most).  Where the look finds that three parts are to
// compute, it costs its call 4 to 5 us: 1.02 to 1.07 of 50 to 380 us forward over the output of a ReLU, 1.01 to 1.10 backward-data
// of a gradient that is mostly zeros, 1.01 to 1.07 backward-filter of both.  A higher line would spare the small calls these and
// take 0.75 to 0.85 from them where their operands suit.
constexpr double kTwoPartShare = 0.45, kTwoPartWgradShare = 0.25;
inline bool two_parts_pay(double share, double kernel_us, double elements) { return share * kernel_us > 4.5 + 4.0 * elements / 5e6; }
// Share of (output position, tap) pairs that lie inside the image
inline double taps_inside(const Problem &pb)
{
    auto axis = [&](int out, int taps, int in) {
        int64_t n = 0;
        for (int r = 0; r < taps; ++r) {                 // o * stride + r - pad in [0, in)
            const int first = std::max(0, (pb.pad - r + pb.stride - 1) / pb.stride);
            const int last = in - 1 + pb.pad - r < 0 ? -1 : std::min(out - 1, (in - 1 + pb.pad - r) / pb.stride);
            n += std::max(0, last - first + 1);
        }
        return (double)n / ((double)out * taps);
    };
    return axis(pb.P, pb.R, pb.H) * axis(pb.Q, pb.S, pb.W);
}
constexpr size_t kSplitRangeBytes = 6400;       // SplitRanges, of which each column has one

// Bytes from the activations of one step of colgemm_split_kernel to those of the next, in the re-laid copy (rows of Wp positions of
// 32 bytes, planes of plane_bytes, three planes to a channel block): the next column of the taps_r x taps_s taps, the next row,
// the next channel block.  In 64 bits: a block of large planes is close to 2^31 bytes, and backward-data (sign -1, taps against the
// planes' order) adds the taps' extent to it.
struct SplitSteps {
    int64_t s, r, c;
};
CONVNET_HD SplitSteps split_steps(unsigned plane_bytes, int Wp, int taps_r, int taps_s, int sign)
{
    return {sign * 32, sign * (Wp - (taps_s - 1)) * 32, (int64_t)3 * plane_bytes - (int64_t)sign * (((taps_r - 1) * Wp + taps_s - 1) * 32)};
}

// Width, split count and time estimate (us, returned) of the three-part fp32 kernel on tiles of bm rows for one column of
// `steps` steps; `groups` columns share the launch.  The split count decides the order of the sums, so it must not depend on
// how many columns run together: it is chosen for one column, the tile width (which changes no sum) for all of them.
//   Time of a round: steps x matrix time of a tile (six products, 4096 FLOP per clock and CU, about 0.75 of it reached)
//   plus 3 us for the first loads and the stores, which nothing hides with one work-group per CU; `weight` times the former.
//   Splits are powers of two (a coarse grid: small shards of a mini-batch then take the same split and give the same
//   bits), of at least 12 steps.  A split adds the launch that sums the partial outputs and their traffic (about 4.5 MB per us).
inline double split_tile_time(int M, int64_t ncols, int steps, int groups, int bm, double weight, int &bn, int &ksplit)
{
    const int64_t mtiles = ceil_div(M, bm);
    const double out_mb = (double)ncols * M * 4.0 / 1e6;
    // best width for a split count: its time, rounds of 256 work-groups
    auto best_width = [&](int ks, int cols, int &width) {
        const int sps = ceil_div(steps, ks);
        double best = 1e30;
        for (int w : {512, 256, 192, 128}) {
            if ((w == 512) != (bm == 32) || (w < 256 && bm != 128)) continue;
            const int64_t units = mtiles * ((ncols + w - 1) / w) * ceil_div(steps, sps) * cols;
            const double us = (double)((units + 255) / 256) * (sps * weight * bm * w * 16 * 12 / 4096.0 / 0.75 / 2200.0 + 3.0);
            if (us < best) { best = us; width = w; }
        }
        return best;
    };
    double best = 1e30;
    ksplit = 1;
    for (int ks = 1; ks <= 8 && (ks == 1 || steps / ks >= 12); ks *= 2) {
        double us = best_width(ks, 1, bn);
        if (ks > 1) us += 5.0 + (ks + 1) * out_mb / 4.5;
        if (us < best * 0.97) { best = us; ksplit = ceil_div(steps, ceil_div(steps, ks)); }
    }
    best_width(ksplit, groups, bn);
    return best;
}

// The same with the rows of the tile: what pads M least, but many tiles of 32 x 512 compete with the taller ones by time, in
// which they count half again: they move more per matrix instruction (0.72 us a step; 64 x 256 with as much work 0.60).
// 224 filters 1x1 on 116x133x54x45: 7 x 32 rows 334 us a call, 2 x 128 rows 263.  The estimate is that of the least padding,
// to which the rules that compare it with the fp32 kernels are fitted.
inline double pick_split_tile(int M, int64_t ncols, int steps, int groups, int &bm, int &bn, int &ksplit)
{
    bm = least_padding(M);
    const double us = split_tile_time(M, ncols, steps, groups, bm, 1.0, bn, ksplit);
    if (bm > 32 || M <= 32) return us;
    double best = split_tile_time(M, ncols, steps, groups, 32, 1.5, bn, ksplit);
    for (int b : {64, 96, 128}) {
        int bn_b, ks_b;
        const double t = split_tile_time(M, ncols, steps, groups, b, 1.0, bn_b, ks_b);
        if (t < best) { best = t; bm = b; bn = bn_b; ksplit = ks_b; }
    }
    return us;
}

constexpr int kDirectMaxRed = 800;
// Small problems go to the vector units (conv_direct_kernels.h): at most 2^24 multiplications, and chains short enough that
// the pass is bound by launches and latency: reduction elements per wavefront (forward / backward-data, one load each),
// positions per thread (backward-filter, five loads each).
inline bool pick_direct(int op, const Problem &pb)
{
    const int64_t J = (int64_t)pb.N * pb.P * pb.Q, crs = (int64_t)pb.C * pb.R * pb.S;
    if (op == kOpBwdFilter) return J * pb.K * crs <= (1 << 24) && J <= 8192 && crs * ceil_div(pb.K, 4) <= 2048;
    const int64_t cols = op == kOpFwd ? J : (int64_t)pb.N * pb.H * pb.W;
    const int64_t red = (int64_t)(op == kOpFwd ? pb.C : pb.K) * pb.R * pb.S, rows = op == kOpFwd ? pb.K : pb.C;
    return cols * rows * red <= (1 << 24) && red <= kDirectMaxRed && pb.R < (1 << 15) && pb.S < (1 << 15) && ((cols + 63) / 64) * ((rows + 3) / 4) <= 1024;
}

constexpr int64_t kWgradPartLimit = (int64_t)48 << 20;    // bytes of partial sums: what the library's own scratch holds

// Split count and time estimate (us, returned) of the three-part fp32 backward-filter kernel on tiles of bm rows: `nblocks`
// blocks of 16 columns, J positions, `groups` columns in one launch.  One work-group per CU, step_us a step of 32 positions and
// 4 us a round for what nothing hides.  Splits that fill one to four rounds of 256 work-groups, of at least four steps; their
// partial sums are written and read once.
inline double wgrad_split_time(int K, int nblocks, int64_t J, int groups, int64_t out_bytes, int bm, double step_us, int &ksplit)
{
    const int steps = (int)((J + 31) / 32);
    const int64_t tiles = (int64_t)ceil_div(K, bm) * ceil_div(nblocks, 16);
    double best = 1e30;
    ksplit = 1;
    for (int r = 1; r <= 4; ++r) {
        int64_t ks = std::min<int64_t>(256 * r / (tiles * groups), steps / 4);
        ks = std::max<int64_t>(1, std::min<int64_t>(ks, kWgradPartLimit / (out_bytes * groups)));
        const int sps = ceil_div(steps, (int)ks), n = ceil_div(steps, sps);
        const double us = (double)((tiles * n * groups + 255) / 256) * (sps * step_us + 4.0) +
                          (2.0 * n + 1.0) * groups * out_bytes / 4.5e6;
        if (us < best * 0.97) { best = us; ksplit = n; }
    }
    return best;
}

// The same with the rows of the tile: what pads K least, but many tiles of 32 rows compete with the taller ones by time, in
// which a step counts 0.95 + 0.0132 BM us (measured 1.37, 1.79, 2.22 and 2.64 for 32 to 128 rows: the 256 columns are loaded
// and split whatever the rows).  352 filters, 194 channels 3x3 stride 2, 68 x 8 x 24: 11 x 32 rows 105 us a call, 3 x 128 rows
// or 4 x 96 (chosen) 52.  The estimate is that of the least padding and of the matrix time of a step (six products, about 0.7 of it reached), to
// which the rule that compares it with the fp32 kernels is fitted.
inline double pick_wgrad_split(int K, int nblocks, int64_t J, int groups, int64_t out_bytes, int &bm, int &ksplit)
{
    bm = least_padding(K);
    const double us = wgrad_split_time(K, nblocks, J, groups, out_bytes, bm, bm * 256.0 * 32 * 12 / 4096.0 / 0.7 / 2100.0, ksplit);
    if (bm > 32 || K <= 32) return us;
    double best = 1e30;
    for (int b : {32, 64, 96, 128}) {
        int ks_b;
        const double t = wgrad_split_time(K, nblocks, J, groups, out_bytes, b, 0.95 + 0.0132 * b, ks_b);
        if (t < best) { best = t; bm = b; ksplit = ks_b; }
    }
    return us;
}

// LDS bytes of one channel block's window under `bn` consecutive positions (n, oh, ow): their padded rows, plus R - 1 more for
// each sample that begins among them, from a multiple of 16 positions on
inline int64_t window_bytes(int N, int OH, int OW, int R, int hp, int wp, int bn, int unit)
{
    const int64_t rows = (bn + OW - 2) / OW + 1, begins = (rows + OH - 2) / OH;
    const int64_t span = std::min<int64_t>(rows + (R - 1) * (begins + 1), (int64_t)N * hp);
    return round_up64((span * wp + 15) * 32, unit);
}

// bf16, stride 1, what the direct-to-LDS kernel does not take: more than 32 rows, more than one block of 16 channels, enough
// taps that the window is worth loading, and a window that fits; and an estimate below that of the register-staged kernel,
// which splits the reduction and so wins where few tiles meet a long one.  Both estimates (us, all columns of a launch
// together: two columns of 48 -> 128 channels at N = 64 are one round of windows and three of the staged kernel) were fitted to
// 280 passes of drawn layers, and looked at again on 700 others that the kernel can take:
//   - several chunks: one work-group of eight waves per CU, whatever its LDS (its registers);
//   - one chunk: two of four waves in 80 KB of LDS, else one, which then has nobody beside it and takes 1.3 times as long a
//     slice (4 x 64 x 19 x 49, two columns of 167 filters 9x9: 51 us, staged 38).
// The rule takes 0.85 of the register-staged kernel's time over those 700, the better of the two each time would take 0.82; of
// the 358 passes that it sends here 13 are 3 to 10 % slower, and of 434 further ones 16, by up to 21 %: where the estimate of
// the register-staged kernel is off (it is good to 17 %; constants fitted anew do no better).  Measured on both sides of the
// line, window / staged: 58 x 80 x 21 x 28, 64 channels 3x3 19 / 32 us; 27 x 112 x 44 x 36, 125 filters 5x5 50 / 72; 8 x 208 x
// 16 x 25, 295 filters 5x5 57 / 56; 7 x 208 x 24 x 14, 144 filters 7x7 95 / 77; 1 x 128 x 14 x 12, 80 filters 5x5 32 / 19.
inline void plan_window(int op, const Problem &pb, Plan &pl)
{
    const bool fwd = op == kOpFwd;
    const int Cr = fwd ? pb.C : pb.K, RS = pb.R * pb.S;
    if (pb.dtype != kDtypeBf16 || op == kOpBwdFilter || pb.stride != 1 || pl.dma || Cr % kChunk != 0 || Cr < 32 || pl.M <= 32 ||
        RS < 9 || pb.S < 3 || (pb.groups > 1 && !pl.fused_groups))
        return;
    const int OH = fwd ? pb.P : pb.H, OW = fwd ? pb.Q : pb.W;
    const int ph = fwd ? pb.pad : pb.R - 1 - pb.pad, pw = fwd ? pb.pad : pb.S - 1 - pb.pad;
    if (ph < 0 || pw < 0) return;
    const int64_t hp = (int64_t)OH + pb.R - 1, wp = (int64_t)OW + pb.S - 1;
    const int G = pb.groups > 1 ? pb.groups : 1;
    const int cb = Cr / 16, ncb = round_up(cb, 3) <= round_up(cb, 2) ? 3 : 2, cbp = round_up(cb, ncb);
    const bool multi = cbp > ncb;
    const int bm = pl.M <= 64 ? 64 : 128, mtiles = ceil_div(pl.M, bm);
    const int64_t ncols = (int64_t)pb.N * OH * OW, xb_bytes = (int64_t)G * cbp * pb.N * hp * wp * 32;
    const int64_t wt_bytes = (int64_t)G * cbp * RS * mtiles * bm * 32;
    if (xb_bytes + (1 << 20) >= kMaxSpanBytes || wt_bytes >= kMaxSpanBytes) return;
    // an odd count of taps: the second group of waves reads a tap past the last, in the row behind the window (unused)
    const int64_t row_behind = multi && RS % 2 ? wp * 32 : 0;
    int64_t best = -1;
    // (six windows of three blocks beside the filters: 8 KB each for 128 rows, 16 for 64, which 192 or 384 positions and their
    // borders fill only in tensors where the narrower tile takes less)
    for (int tn = multi && ncb == 3 ? 2 : 3; tn >= 2; --tn) {
        const int bn = tn * 32 * (bm == 64 ? 4 : 2);
        const int64_t win = window_bytes(pb.N, OH, OW, pb.R, (int)hp, (int)wp, bn, multi ? 8192 : 1024);   // (a round of loads)
        int64_t lds = (multi ? 6 : 2) * (int64_t)ncb * bm * 32 + (multi ? 2 : 1) * ncb * win;
        if (multi) lds = std::max<int64_t>(lds, 8 * tn * 4096);          // the sums that the two groups of waves trade
        // (a round of every block per step, none in a chunk's last two steps)
        if (lds + row_behind > 160 * 1024 || (multi && win / 8192 > (RS + 1) / 2 - 2)) continue;
        const int64_t tiles = mtiles * ((ncols + bn - 1) / bn) * G, per_round = !multi && lds <= 80 * 1024 ? 512 : 256;
        const int64_t cost = (tiles + per_round - 1) / per_round * bn;
        if (best >= 0 && cost >= best) continue;
        best = cost;
        pl.win_tn = tn; pl.win_bytes = (int)win; pl.win_lds = (int)lds;
    }
    if (best < 0) return;
    {
        const int bn = pl.win_tn * 32 * (bm == 64 ? 4 : 2), slots = !multi && pl.win_lds <= 80 * 1024 ? 512 : 256;
        const int64_t tiles = mtiles * ((ncols + bn - 1) / bn) * G, rounds = (tiles + slots - 1) / slots;
        const double slices = cbp * RS * (pl.win_tn == 3 ? 1.0 : 0.72);
        const bool lone = !multi && slots == 256;
        const double us = (lone ? 9.5 : 11.7) + 0.6 * xb_bytes / 1e6 +
                          (multi  ? 0.148 * slices * rounds
                           : lone ? 0.17 * slices * (tiles > 256 ? 1.2 * rounds : 1.0)
                                  : 0.131 * slices * (tiles > 256 ? 2 * rounds : 1));
        const int kc = Cr % 64 == 0 ? 64 : Cr % 48 == 0 ? 48 : Cr % 32 == 0 ? 32 : 16;           // channels per step
        const int64_t staged = (pl.Mpad / pl.tile.bm()) * ((ncols + pl.tile.bn() - 1) / pl.tile.bn()) * pl.nsplit * G;
        const double steps = (double)ceil_div(Cr / kc * RS, pl.nsplit) * ((staged + 255) / 256);
        const double staged_us = 12.5 + 0.33 * pl.blk_bytes / 1e6 +
                                 (pl.nsplit > 1 ? 3.1 + 0.26 * ncols * G * pl.M * 4.0 * pl.nsplit / 1e6 : 0.0) +
                                 steps * (0.0943 * kc / 16 * pl.tile.bm() * pl.tile.bn() / 16384.0 + 0.14);
        if (us >= 0.9 * staged_us) return;
    }
    pl.win = true;
    pl.win_lds += (int)row_behind;
    pl.win_bm = bm; pl.win_ncb = ncb; pl.win_cb = cbp; pl.win_hp = (int)hp; pl.win_wp = (int)wp; pl.win_ph = ph; pl.win_pw = pw;
    pl.nsplit = 1;
    pl.wt_off = 0; pl.wt_bytes = (size_t)wt_bytes;
    pl.xb_off = round_up64(wt_bytes, 256);
    // the last tiles' windows and the filters past the last step reach behind the tensors
    pl.xb_bytes = (size_t)xb_bytes + 2 * (size_t)pl.win_bytes + 6 * (size_t)ncb * mtiles * bm * 32;
    pl.total = pl.xb_off + round_up64(pl.xb_bytes, 256);
}

// LDS layout of the first-layer backward-filter in three parts (wgrad_rows_split_kernel).  A staged input row holds its parts one
// after the other and zeros behind them: an output row is read in whole blocks of 16 positions, and the last of four blocks
// reaches past the third part, where the next row of the ring may be being staged.
constexpr int kRowsSplitThreads = 512;
constexpr int kRowsSplitPitch = 456;                              // bytes of a part: 228 padded input columns
constexpr int kRowsSplitGap = 72;
constexpr int kRowsSplitRow = 3 * kRowsSplitPitch + kRowsSplitGap;
// one past the last byte of a part's row that the reads of `blocks` blocks touch: two quads of eight bytes at every position, from
// position 8 half + 0..3 and quad sg = 0..2 of a filter row on, the second 32 bytes behind the first
constexpr int rows_split_read_end(int blocks) { return (blocks - 1) * 128 + (8 + 3 + 2) * 8 + 32 + 8; }

// three_part = false: the kernels that want the least workspace: fp32 passes on the fp32 kernels, no input windows, the columns of
// a grouped bf16 backward-filter one after the other
inline Plan make_plan(int op, const Problem &pb, bool three_part = true)
{
    Plan pl = {};
    pl.op = op;
    pl.direct = pick_direct(op, pb);
    const int G = pb.groups > 1 ? pb.groups : 1;
    const int RS = pb.R * pb.S;
    if (op == kOpFwd) { pl.M = pb.K; pl.Kg = pb.C * RS; }
    else if (op == kOpBwdData) { pl.M = pb.C; pl.Kg = pb.K * RS; }
    else { pl.M = pb.K; pl.Kg = pb.C * RS; }
    pl.tile = pick_tile(pl.M);
    {
        // bf16 inputs, at least 97 GEMM rows, gathered channel count a multiple of 32: the direct-to-LDS kernel
        const bool fwd = op == kOpFwd;
        const int Cg = fwd ? pb.C : pb.K;
        if (pb.dtype == kDtypeBf16 && G == 1 && (fwd || (op == kOpBwdData && pb.stride == 1)) && Cg % 32 == 0 &&
            pl.M > 96) {
            const int OH = fwd ? pb.P : pb.H, OW = fwd ? pb.Q : pb.W, mul = fwd ? pb.stride : 1;
            const int ph = fwd ? pb.pad : pb.R - 1 - pb.pad, pw = fwd ? pb.pad : pb.S - 1 - pb.pad;
            const int64_t hp = (int64_t)(OH - 1) * mul + pb.R, wp = (int64_t)(OW - 1) * mul + pb.S;
            const int64_t bytes = (int64_t)pb.N * (Cg / 16) * hp * wp * 32;
            if (ph >= 0 && pw >= 0 && bytes < kMaxSpanBytes) {
                pl.dma = true;
                pl.dma_hp = (int)hp; pl.dma_wp = (int)wp; pl.dma_ph = ph; pl.dma_pw = pw;
                const int64_t ncols = (int64_t)pb.N * OH * OW;
                pick_dma_tile(Cg, ceil_div(pl.M, 128), ncols, pl.tile, pl.dma_kc, pl.dma_occ);
                pl.xb_bytes = (size_t)bytes;
            }
        }
    }
    if (!pl.dma) {
        // 33..48 rows on the fp32 fast path: 16 x 16 matrix blocks instead of padding to 64 rows
        const int Cg = op == kOpFwd ? pb.C : pb.K;
        if (pb.dtype == kDtypeF32 && pl.M > 32 && pl.M <= 48 && Cg % kChunk == 0 &&
            (op == kOpFwd || (op == kOpBwdData && pb.stride == 1)))
            pl.tile = kTile48x256;
    }
    pl.Mpad = round_up(pl.M, pl.tile.bm());
    pl.Kgpad = round_up(pl.Kg, kChunk);
    pl.tab_len = round_up(pl.Kg + 2 * kChunk, kTapTablePad);   // two steps of slack for the prefetch
    pl.kc = kChunk;
    pl.nsplit = 1;
    pl.chunks_per_split = 0;
    double fp32_us = 0;                            // forward / backward-data: estimated time of one column in fp32
    size_t off = 0;
    pl.tab_off = off; pl.tab_bytes = (size_t)pl.tab_len * 16; off += round_up64(pl.tab_bytes, 256);
    if (op == kOpBwdFilter) {
        const int64_t J = (int64_t)pb.N * pb.P * pb.Q;
        const int jchunks = (int)((J + kChunk - 1) / kChunk);
        pl.fused_groups = G > 1 && pb.dtype == kDtypeF32 && pb.C % kChunk == 0;
        const int tiles = (pl.Mpad / pl.tile.bm()) * ceil_div(pl.Kg, pl.tile.bn()) * (pl.fused_groups ? G : 1);
        // as many splits as fill two work-groups per CU without exceeding them
        int want = kTargetGroups / tiles;
        int most = jchunks / 8 > 0 ? jchunks / 8 : 1;     // at least 8 chunks of work per split
        int nsplit = want < most ? want : most;
        if (nsplit < 1) nsplit = 1;
        pl.chunks_per_split = ceil_div(jchunks, nsplit);
        pl.nsplit = ceil_div(jchunks, pl.chunks_per_split);
        if (pb.dtype == kDtypeBf16 && pb.C % kChunk == 0 && pl.tile.bn() == 128 && pb.stride == 1 &&
            pb.P == pb.H && pb.Q == pb.W && pb.R - 1 == 2 * pb.pad && pb.S - 1 == 2 * pb.pad) {
            const int wq = pb.W + pb.pad;
            const int jy = round_up(pb.P * wq, 8);
            const int jx = round_up(jy + (pb.R - 1) * wq + pb.S, 8);
            const int64_t steps = ((int64_t)pb.N * jy + 63) / 64;
            // (x is packed twice: the second copy, moved up by one element, serves the taps with an odd shift)
            // (dy is packed step-major with its rows padded to whole 128-row tiles: the direct-to-LDS kernel, one
            // work-group of 128 x 256 per CU)
            const int kpad = round_up(pb.K, 128);
            const int64_t dy_bytes = (int64_t)kpad * steps * 64 * 2, x_bytes = (int64_t)2 * pb.C * pb.N * jx * 2;
            if (jy >= 64 && dy_bytes < kMaxSpanBytes && x_bytes < kMaxSpanBytes) {
                // splits of the reduction that fill the CUs once, of at least four steps; returned: steps one after the other on a CU
                const int tiles1 = (kpad / 128) * ceil_div(pl.Kg, 256);
                auto pick_splits = [&](int columns, int &per_split, int &nsplit_) {
                    const int ns = std::max(1, std::min(256 / (tiles1 * columns), (int)(steps / 4)));
                    per_split = ceil_div((int)steps, ns);
                    nsplit_ = ceil_div((int)steps, per_split);
                    return (double)per_split * (((int64_t)tiles1 * nsplit_ * columns + 255) / 256);
                };
                // The columns of a grouped layer in one launch of each kernel, where their packed copies together can still be
                // indexed: it saves about 14 us a further column, and costs about 0.6 us for each step that a CU does more of
                // than apart, where whole tiles of all columns leave no splits to even out the CUs.  Long reductions gain
                // nothing, and lose where the copies of all columns, read once a tap, are more than the 256 MB cache holds
                // beside what passes through it (a 1x1 layer reads them once).  Apart / together, us: two columns of 48 -> 128
                // channels 5x5, N = 16 56 / 30, 64 78 / 60, 128 120 / 100, 192 162 / 157, 208 (156 MB) 171 / 170, 240 191 / 195;
                // two of 160 -> 384 7x7 on 17x24, N = 71, 515 steps either way 437 / 422; two of 496 -> 512 3x3 on 38x32, N = 42,
                // 825 steps for 550 624 / 957; three of 304 -> 384 5x5 on 30x16, N = 134, 2278 for 1710 1485 / 2842.  Over 212
                // layers of two to eight columns this takes 0.83 of their time apart (always together 1.04).
                int per1, n1, per_all, n_all;
                const double apart = G * pick_splits(1, per1, n1), all = pick_splits(G, per_all, n_all);
                pl.fused_groups = G > 1 && three_part && dy_bytes * G < kMaxSpanBytes && x_bytes * G < kMaxSpanBytes &&
                                  (RS == 1 || (dy_bytes + x_bytes) * G < (int64_t)155000000) && all <= 200.0 &&
                                  0.6 * (all - apart) < 14.0 * (G - 1);
                const int GF = pl.fused_groups ? G : 1;
                pl.lin = true;
                pl.lin_wq = wq; pl.lin_jy = jy; pl.lin_jx = jx; pl.lin_steps = (int)steps;
                pl.chunks_per_split = pl.fused_groups ? per_all : per1;
                pl.nsplit = pl.fused_groups ? n_all : n1;
                pl.lin_dy_off = off; pl.lin_dy_bytes = (size_t)dy_bytes * GF; off += round_up64(pl.lin_dy_bytes, 256);
                pl.lin_x_off = off; pl.lin_x_bytes = (size_t)x_bytes * GF; off += round_up64(pl.lin_x_bytes, 256);
            }
        }
        pl.part_off = off;
        const bool staged = pb.C % kChunk == 0;          // fast path always goes through the partials
        pl.part_bytes = (pl.nsplit > 1 || staged) ? (size_t)pl.nsplit * pb.K * pb.C * RS * 4 : 0;
        if (pb.dtype == kDtypeBf16 && G == 1 && pb.stride == 4 && pb.pad == 2 && pb.S <= 11 && pb.R <= 12 &&
            pb.C <= 4 && pl.Kg <= 384 && pb.K <= 96 && pb.Q <= 64 && pb.W % 8 == 0 && pb.x_bs % 8 == 0) {
            const int lds = 2 * 96 * 144 + pb.C * 16 * pb.S * 144 + (255 * 16 + 10 * 144 + 16);   // + trash area
            if (lds <= 150 * 1024) {
                pl.rows = true;
                pl.rows_lds = lds;
                int splits = ceil_div(256, pb.N);
                if (splits > pb.P) splits = pb.P;
                pl.rows_splits = splits;
                const int64_t units = (int64_t)pb.N * splits;
                pl.rows_wgs = units < 256 ? (int)units : 256;
                const size_t need = (size_t)pl.rows_wgs * pb.K * pl.Kg * 4;
                if (need > pl.part_bytes) pl.part_bytes = need;     // the table path stays available at run time
            }
        }
        if (pb.dtype == kDtypeF32 && G == 1 && pb.C <= 4 && pb.K > 48 && pb.K <= 96 && pl.Kg > 128 && pl.Kg <= 384 &&
            pb.Q <= 57 && pb.R + pb.stride <= 16 && pb.stride <= 4 && pb.W <= 256) {
            int wp = pb.W + 2 * pb.pad;                      // pitch = 48 mod 64: taps of up to four filter rows
            wp += (48 - wp % 64 + 64) % 64;                  // read by one wave fall into different banks
            const int64_t lds = ((int64_t)2 * 96 * 58 + (int64_t)pb.C * 16 * wp + 64) * 4;   // + slack
            if (lds <= 150 * 1024) {
                pl.rows_f32 = true;
                pl.rows_lds = (int)lds;
                pl.rows_wp = wp;
                int splits = ceil_div(256, pb.N);
                if (splits > pb.P) splits = pb.P;
                pl.rows_splits = splits;
                const int64_t units = (int64_t)pb.N * splits;
                pl.rows_wgs = units < 256 ? (int)units : 256;
                pl.part_bytes = (size_t)pl.rows_wgs * pb.K * pl.Kg * 4;
                // Three parts: stride 4 (a quad of taps is then eight aligned bytes of a staged row), 13 blocks of 32 columns,
                // rows of 228 staged columns.  An output row costs it 60 matrix instructions of 32 clocks per SIMD for each
                // block of 16 positions (two waves of 30), and the fp32 kernel 9 of 64 for each pair of positions: 2.4 times
                // as much in full blocks, less in rows of up to six.  Its start (149 KB of LDS to clear, a wave's worth of
                // tables) is 9 us longer.  Fitted to 126 drawn layers: 28 us, 0.27 a row and 1.09 a block of it, against 19
                // us, 1.13 a row and 0.26 a pair.  With the line at 10 us they take 1.001 times what the better of the two
                // each time would, and none that it sends here took longer (three parts / fp32, us, rows per work-group:
                // 1 position, 20 rows 56 / 51; 4, 26 rows 62 / 64; 7, 22 rows 55 / 60; 16, 6 rows 34 / 36; 33, 6 rows
                // 51 / 53; 55, 10 rows 81 / 102; first layer N = 16 53.5 / 56.8, N = 300 569 / 954).
                const int quads = pb.C * pb.R * ceil_div(pb.S, 4), blocks = ceil_div(pb.Q, 16);
                const int rows = (int)((units + pl.rows_wgs - 1) / pl.rows_wgs) * ceil_div(pb.P, splits);    // per work-group
                // staging items of four values, two of x and three of dy per thread.  (The conditions below leave at most 3 x 4 x
                // 57 and 96 x 14 of them: with four channels the input rows would not fit the LDS.)
                const int x_items = pb.C * std::min(pb.R, 4) * (pb.Q - 1 + ceil_div(pb.S, 4)), dy_items = pb.K * ceil_div(pb.Q, 4);
                const int64_t split_lds = 2 * 3 * 96 * 144 + (int64_t)pb.C * 16 * kRowsSplitRow;
                if (three_part && pb.stride == 4 && pb.S <= 12 && quads <= 104 && pb.Q <= 55 && split_lds <= 150 * 1024 &&
                    x_items <= 2 * kRowsSplitThreads && dy_items <= 3 * kRowsSplitThreads &&
                    (int64_t)pb.N * pb.P >= 3 * 256 && rows * (0.85 + 0.26 * ceil_div(pb.Q, 2) - 1.09 * blocks) > 10.0) {
                    pl.rows_split = true;
                    pl.rows_lds = (int)split_lds;
                }
            }
        }
        off += round_up64(pl.part_bytes * (pl.fused_groups ? G : 1), 256);
    } else {
        const int Cr_ = op == kOpFwd ? pb.C : pb.K;
        // (fp32 kernels, and the bf16 kernel that stages through registers: neither widens nor takes the direct-to-LDS path)
        pl.fused_groups = G > 1 && (pb.dtype == kDtypeF32 || pb.dtype == kDtypeBf16) && Cr_ % kChunk == 0 &&
                          (op == kOpFwd || pb.stride == 1) && !pl.dma;
        const int GF = pl.fused_groups ? G : 1;
        pl.wt_off = off;
        pl.wt_bytes = (size_t)pl.Mpad * pl.Kgpad * 4;
        off += round_up64(pl.wt_bytes * GF, 256);
        // Fast path (channel count of the gathered tensor a multiple of 16, unit-stride gather rows):
        // the reduction may be cut into ranges when that balances the CUs better.  Model: a CU
        // holding c work-groups runs them at eff(c) of its MFMA rate; the launch lasts as long
        // as its fullest CU; the partial outputs cost one extra pass over memory per range.
        const int Cr = op == kOpFwd ? pb.C : pb.K;
        const int OH = op == kOpFwd ? pb.P : pb.H, OW = op == kOpFwd ? pb.Q : pb.W;
        if (Cr % kChunk == 0 && (op == kOpFwd || pb.stride == 1) && !pl.dma) {
            const int64_t ncols = (int64_t)pb.N * OH * OW;
            // measured fraction of the MFMA rate a CU reaches with c resident work-groups
            const double eff16[5] = {1.0, 0.71, 0.83, 0.87, 0.88};
            // time of `cols` columns in one launch, and the split that gives it
            // (32-deep steps were measured too: no faster at two work-groups per CU, so steps stay 16 deep)
            auto best_split = [&](int cols, int &nsplit, int &per_split) {
                const int tiles = (pl.Mpad / pl.tile.bm()) * (int)((ncols + pl.tile.bn() - 1) / pl.tile.bn()) * cols;
                const double out_mb = (double)ncols * pl.M * 4.0 * cols / 1e6;
                const int steps = (Cr / kChunk) * RS;
                const double step_us = pl.tile.bm() * pl.tile.bn() * 2.0 * kChunk / 64.0 / 4.0 / 2100.0;   // MFMA time
                double best = 1e30;
                for (int ks = 1; ks <= 4; ++ks) {
                    if (ks > 1 && steps * kChunk / ks < 256) break;
                    const int sps = ceil_div(steps, ks);
                    const int units = tiles * ceil_div(steps, sps);
                    const int per_cu = ceil_div(ceil_div(units, 8), 32);
                    const int resident = per_cu < 4 ? per_cu : 4;
                    double us = per_cu * sps * step_us / eff16[resident];
                    if (ks > 1) us += 5.0 + (ks + 1) * out_mb / 4.5;      // launch + partial traffic at ~4.5 MB/us
                    if (us < best * 0.97) { best = us; nsplit = ceil_div(steps, sps); per_split = sps; }
                }
                return best;
            };
            int ns1, ps1;
            fp32_us = best_split(1, ns1, ps1);
            best_split(GF, pl.nsplit, pl.chunks_per_split);
            if (pl.nsplit > 1) {
                pl.part_off = off;
                pl.part_bytes = (size_t)pl.nsplit * ncols * pl.M * 4;
                off += round_up64(pl.part_bytes * GF, 256);
            }
        }
        if (pl.chunks_per_split == 0) pl.chunks_per_split = pl.Kgpad / kChunk;
    }
    // bf16 inputs go straight to the bf16 MFMA kernels where the gathered channel count is a multiple of 16
    // (backward-filter: 128-column tiles only).  The few-channel kernels (patch forward, table backward-filter)
    // read bf16 tensors themselves and only want fp32 filters; every other shape is widened to dense fp32
    // copies, batch strides dropped, and takes the fp32 kernels.
    const int Cr = op == kOpBwdData ? pb.K : pb.C;
    const bool bf16_kernel = Cr % kChunk == 0 &&
        (op == kOpFwd || (op == kOpBwdData && pb.stride == 1) || (op == kOpBwdFilter && pl.tile.bn() == 128));
    if (op == kOpFwd && !(pb.C % kChunk == 0)) {
        const int tm = pl.M <= 32 ? 1 : pl.M <= 64 ? 2 : pl.M <= 96 ? 3 : 4;
        const int bm = tm * 32, mpad = round_up(pl.M, bm);
        int span = (pb.Q + 126) / pb.Q;                 // output rows a 128-position tile can straddle, minus one
        if (span > pb.P - 1) span = pb.P - 1;
        const int nr = span * pb.stride + pb.R;
        const int need_w = pb.W + 2 * pb.pad > (pb.Q - 1) * pb.stride + pb.S ? pb.W + 2 * pb.pad
                                                                              : (pb.Q - 1) * pb.stride + pb.S;
        const int wp = round_up(need_w, 4);
        const int64_t lds64 = ((int64_t)2 * bm * 20 + pl.Kgpad + (int64_t)pb.C * nr * wp) * 4;
        if (lds64 <= 80 * 1024 && (int64_t)mpad * pl.Kgpad * 4 <= (int64_t)pl.wt_bytes) {
            pl.patch = true;
            pl.patch_tm = tm; pl.patch_nr = nr; pl.patch_wp = wp; pl.patch_lds = (int)lds64;
        }
    }
    const bool bf16_in = pb.dtype == kDtypeBf16;
    const bool direct = pl.patch || (op == kOpBwdFilter && pb.C % kChunk != 0);   // kernels that read bf16 themselves
    pl.widen = bf16_in && !bf16_kernel && !direct;
    pl.widen_w = bf16_in && !bf16_kernel && op != kOpBwdFilter;
    if (pl.dma) {
        pl.xb_off = off;
        off += round_up64(pl.xb_bytes, 256);
    } else if (pb.dtype == kDtypeBf16 && bf16_kernel && op != kOpBwdFilter) {
        pl.blk_off = off;
        pl.blk_bytes = (size_t)pb.N * Cr * (pl.fused_groups ? G : 1) * (op == kOpFwd ? pb.H * pb.W : pb.P * pb.Q) * 2;
        off += round_up64(pl.blk_bytes, 256);
    }
    if (pb.out_bf16 && op != kOpBwdFilter && !bf16_kernel && !pl.patch) {
        pl.stage_off = off;
        pl.stage_bytes = (size_t)pb.N * (op == kOpFwd ? (size_t)pb.K * pb.P * pb.Q : (size_t)pb.C * pb.H * pb.W) * 4;
        off += round_up64(pl.stage_bytes, 256);
    }
    if (pl.widen || pl.widen_w) {
        const int64_t x_e = (int64_t)pb.N * pb.C * pb.H * pb.W, y_e = (int64_t)pb.N * pb.K * pb.P * pb.Q;
        const int64_t w_e = (int64_t)pb.K * pb.C * RS;
        // slot 0: the activation-side input; slot 1: the filters (forward, backward-data) or dy (backward-filter)
        const int64_t a = op == kOpBwdData ? y_e : x_e;
        const int64_t b = op == kOpBwdFilter ? y_e : w_e;
        const bool need0 = pl.widen, need1 = op == kOpBwdFilter ? pl.widen : pl.widen_w;
        pl.cvt_off[0] = off; pl.cvt_bytes[0] = need0 ? (size_t)a * 4 : 0; off += round_up64(pl.cvt_bytes[0], 256);
        pl.cvt_off[1] = off; pl.cvt_bytes[1] = need1 ? (size_t)b * 4 : 0; off += round_up64(pl.cvt_bytes[1], 256);
    }
    pl.total = off;

    // fp32 forward / stride-1 backward-data through the bf16 matrix instruction, where that is estimated to be faster
    // than the fp32 kernels: it needs a pass over the input (4 bytes read, 6 written per padded position and channel)
    // that layers with little work per input element do not earn back.  The estimate is per column, so that a grouped
    // layer takes the route its columns would take alone.
    if (three_part && !pl.direct && pb.dtype == kDtypeF32 && (op == kOpFwd || (op == kOpBwdData && pb.stride <= 4)) &&
        (Cr >= 16 || (op == kOpFwd && pb.stride <= 4 && Cr * pb.stride * pb.stride >= 16))) {
        const bool fwd = op == kOpFwd, strided = !fwd && pb.stride > 1;
        const int GF = pl.fused_groups ? G : 1;
        // forward: folding pads the filter to whole strides but leaves fewer channels to pad to blocks of 16
        const int f = pb.stride;
        const bool shorter = f > 1 && f <= 4 && ceil_div(Cr * f * f, 16) * ceil_div(pb.R, f) * ceil_div(pb.S, f) < ceil_div(Cr, 16) * RS;
        const int fold = pl.sp_fold = fwd && shorter && !pl.fused_groups ? f : 1;
        const int R = ceil_div(pb.R, fold), S = ceil_div(pb.S, fold), RS_ = R * S;
        const int OH = fwd ? pb.P : pb.H, OW = fwd ? pb.Q : pb.W, mul = fwd && fold == 1 ? pb.stride : 1;
        // zero rows before the data, rows of the padded planes; strided: dy rows -(taps - 1) .. (H - 1 + pad) / stride
        const int rtaps = ceil_div(pb.R, pb.stride), staps = ceil_div(pb.S, pb.stride);
        pl.sp_ph = fwd ? pb.pad : strided ? rtaps - 1 : pb.R - 1 - pb.pad;
        pl.sp_pw = fwd ? pb.pad : strided ? staps - 1 : pb.S - 1 - pb.pad;
        const int64_t hp = strided ? (pb.H - 1 + pb.pad) / pb.stride + rtaps : (int64_t)(OH - 1) * mul + R;
        const int64_t wp = strided ? (pb.W - 1 + pb.pad) / pb.stride + staps : (int64_t)(OW - 1) * mul + S;
        const int cb = ceil_div(Cr * fold * fold, 16);
        const int64_t ncols = (int64_t)pb.N * OH * OW;
        const int steps = strided ? ceil_div(cb * RS, pb.stride * pb.stride) : cb * RS_;      // strided: mean over the classes
        int bm, bn, ks;
        double us = pick_split_tile(pl.M, ncols, steps, GF, bm, bn, ks);
        const double tile_us = us;
        us += 2.0 + ((double)pb.N * Cr * (fwd ? pb.H * pb.W : pb.P * pb.Q) * 4.0 + (double)pb.N * cb * hp * wp * 96.0) / 3.8e6;
        // a stride beyond the filter: most positions get a zero, and the stores, every stride-th word of a row, decide
        // (192 channels at 89x35x31, 51 filters 1x1 stride 3: 71 us, fp32 44; 224 at 100x29x39, 96 filters stride 2: 88, 120)
        const bool gaps = strided && (pb.R < pb.stride || pb.S < pb.stride);
        if (gaps) us = std::max(us, 14.5 + 0.64 * ncols * pl.M * 4.0 / 1e6);
        // the few-channel kernel reaches about 90 TFLOP/s on its padded rows, at 1 us or more per 16-deep step; the
        // tap-table kernel 55 and 1.7 us
        const double gflop = 2.0 * ncols * Cr * RS / 1e9;          // per row
        if (pl.patch)
            fp32_us = std::max(gflop * round_up(pl.M, 32) / 90.0 * 1e3, 1.0 * ceil_div(Cr * RS, kChunk)) + 3.0;
        else if (gaps)
            fp32_us = std::max(gflop * pl.M / 38.0 * 1e3 + 8.0, 15.0 + 1.2 * ceil_div(Cr * RS, kChunk));
        else if (strided)              // all taps at every position, masked: 20 TFLOP/s of them
            fp32_us = std::max(gflop * pl.M / 20.0 * 1e3, 1.7 * ceil_div(Cr * RS, kChunk));
        else if (Cr % kChunk != 0)
            fp32_us = std::max(gflop * pl.M / 55.0 * 1e3, 1.7 * ceil_div(Cr * RS, kChunk));
        const int mpad = round_up(pl.M, bm);
        const int64_t x_bytes = (int64_t)pb.N * GF * cb * hp * wp * 96, w_bytes = (int64_t)GF * cb * RS_ * mpad * 96;
        const int64_t limit = (int64_t)1 << 32;      // 32-bit byte offsets
        // (one product: the fp32 kernels round it once, the six products leave out up to 2^-23 of it; from two on the error of
        // the fp32 kernels is the larger one)
        if (us * 1.1 < fp32_us && (int64_t)Cr * RS > 1 && pl.sp_ph >= 0 && pl.sp_pw >= 0 && x_bytes < limit && w_bytes < limit / 2) {
            pl.sp = true;
            pl.sp_bm = bm; pl.sp_bn = bn; pl.sp_cb = cb; pl.sp_hp = (int)hp; pl.sp_wp = (int)wp; pl.sp_mpad = mpad;
            pl.chunks_per_split = ceil_div(steps, ks);
            pl.nsplit = ceil_div(steps, pl.chunks_per_split);
            // More than two rounds of tiles with short reductions: half the width on four waves, two work-groups to a CU, so that
            // one's first loads and stores pass under the other's matrix instructions (whole layers, 8 -> 4 waves: 128 x 3 x 224 x
            // 224, 96 filters 11x11, 27 steps 404 -> 397 us; two columns 48 -> 128 5x5, 75 and 100 steps 1069 -> 1077).  On 91
            // drawn passes up to the line it takes 0.80 to 1.02 of the wider tiles' time, 0.92 in the mean; on 57 beyond it
            // 0.89 to 1.04: the line is where it stops losing nowhere.  In one round it costs more: 384 -> 384 3x3, kernel 231
            // -> 241, 384 -> 256 172 -> 213.
            if (bn == 256 && pl.chunks_per_split <= 45 && (int64_t)(mpad / bm) * ((ncols + 255) / 256) * pl.nsplit * GF > 512) {
                pl.sp_pair = true;
                pl.sp_bn = 128;
            }
            pl.sp_w_off = 0; pl.sp_w_bytes = (size_t)w_bytes;
            pl.sp_x_off = round_up64(w_bytes, 256); pl.sp_x_bytes = (size_t)x_bytes;
            pl.part_off = pl.sp_x_off + round_up64(x_bytes, 256);
            pl.part_bytes = pl.nsplit > 1 ? (size_t)pl.nsplit * ncols * pl.M * 4 : 0;
            pl.total = pl.part_off + round_up64(pl.part_bytes * GF, 256);
            const int least = strided ? cb * (pb.R / pb.stride) * (pb.S / pb.stride) / pl.nsplit : pl.chunks_per_split;
            // of the positions and taps that the pass goes over (backward-data: a share 1 / stride^2 of the taps at each)
            const double inside =
                taps_inside(pb) * (fwd ? 1.0 : (double)pb.P * pb.Q * pb.stride * pb.stride / ((double)pb.H * pb.W));
            const float dense = (float)(std::min(inside, 1.0) * Cr * RS / (16.0 * cb * (strided ? RS : RS_)));
            // (the four-wave kernels read three parts: without this their 45 steps would have to stay below what two parts begin at)
            // (and a preparing work-group's 128 positions lie in four columns at most: 47 steps are as many positions and more)
            if (!pl.sp_pair && (GF <= 4 || cb * hp * wp >= 43) && split_segments(dense, false, least) > 0 &&
                two_parts_pay(kTwoPartShare, tile_us, (double)pb.N * Cr * (fwd ? pb.H * pb.W : pb.P * pb.Q) + (double)pb.K * pb.C * RS)) {
                pl.sp_two = true;
                pl.sp_two_steps = least;
                pl.sp_dense = dense;
                pl.sp_range_off = pl.total;
                pl.sp_range_bytes = kSplitRangeBytes * GF;
                pl.total += pl.sp_range_bytes;
            }
        }
    }
    // fp32 backward-filter through the bf16 matrix instruction, where that is estimated to be faster than the fp32 kernels
    // (few-channel layers pad 16 / C times) and its partial sums fit where theirs do.
    if (three_part && !pl.direct && pb.dtype == kDtypeF32 && op == kOpBwdFilter && pb.K >= 8 && pb.C >= 8 &&
        std::max((int64_t)pb.H * pb.W, (int64_t)pb.P * pb.Q) * 32 < kMaxSpanBytes) {
        const int GF = pl.fused_groups ? G : 1;
        const int64_t J = (int64_t)pb.N * pb.P * pb.Q, out_bytes = (int64_t)pb.K * pl.Kg * 4;
        const int cb = ceil_div(pb.C, 16);
        // fp32 kernels: matrix time of their 16-deep steps, of which the staged kernel reaches about 0.8 with two
        // work-groups per CU, the tap-table kernel 0.5 (and two launches more); few-channel rows 104 TFLOP/s
        // (both estimates are for one column alone, so that a column takes the same route in a grouped layer)
        const double step_us = pl.tile.bm() * (double)pl.tile.bn() * 32.0 / 256.0 / 2100.0;
        const int tiles = (pl.Mpad / pl.tile.bm()) * ceil_div(pl.Kg, pl.tile.bn()), jchunks = (int)((J + kChunk - 1) / kChunk);
        const int per_split = ceil_div(jchunks, std::max(1, std::min(kTargetGroups / tiles, jchunks / 8)));
        const int ns = ceil_div(jchunks, per_split);
        fp32_us = (double)(((int64_t)tiles * ns + 255) / 256) * per_split * step_us / (pb.C % kChunk == 0 ? 0.8 : 0.5) + 4.0 +
                  (2.0 * ns + 1.0) * out_bytes / 4.5e6 + (pb.C % kChunk == 0 ? 0.0 : 4.0);
        if (pl.rows_f32) fp32_us = 2.0 * J * pb.K * pl.Kg / 104e6;
        int bm, ks;
        const double us = pick_wgrad_split(pb.K, RS * cb, J, 1, out_bytes, bm, ks);
        pick_wgrad_split(pb.K, RS * cb, J, GF, out_bytes, bm, ks);
        const int64_t part = (int64_t)ks * out_bytes;
        const int steps = (int)((J + 31) / 32);
        if (us * 1.05 + 1.5 < fp32_us && J > 1 && (part * GF <= kWgradPartLimit || part * GF <= (int64_t)pl.total)) {
            pl.sp = true;
            pl.sp_bm = bm; pl.sp_bn = 256; pl.sp_cb = cb;
            pl.chunks_per_split = 2 * ceil_div(steps, ks);       // chunks of 16 positions, two to a step
            pl.nsplit = ceil_div(2 * steps, pl.chunks_per_split);
            pl.part_off = 0; pl.part_bytes = (size_t)pl.nsplit * out_bytes;
            pl.total = round_up64(pl.part_bytes * GF, 256);
            const float dense = (float)taps_inside(pb);
            // (three parts where only their partial sums fit the library's own scratch: a call on that gives the same bits)
            const bool fits = (int64_t)pl.total > kWgradPartLimit || (int64_t)(pl.total + kSplitRangeBytes * GF) <= kWgradPartLimit;
            if (fits && split_segments(dense, false, pl.chunks_per_split) > 0 &&
                two_parts_pay(kTwoPartWgradShare, us, (double)pb.N * (pb.C * pb.H * pb.W + pb.K * pb.P * pb.Q))) {
                pl.sp_two = true;
                pl.sp_dense = dense;
                pl.sp_range_off = pl.total;
                pl.sp_range_bytes = kSplitRangeBytes * GF;
                pl.total += pl.sp_range_bytes;
            }
        }
    }
    if (three_part && !pl.direct) plan_window(op, pb, pl);
    return pl;
}

// A workspace that three parts fit into, but not what the operands' range is found with: three parts
inline void fit_two_parts(Plan &pl, size_t ws_bytes)
{
    if (!pl.sp_two || ws_bytes >= pl.total || ws_bytes < pl.total - pl.sp_range_bytes) return;
    pl.sp_two = false;
    pl.total -= pl.sp_range_bytes;
}

// The plan of a call that brings ws_bytes of workspace.  The three-part kernels want up to six bytes per padded input element,
// the window kernel and the columns of a backward-filter in one launch more than the staged kernel and one column; a caller that
// has less, but as much as those take, gets those.
inline Plan plan_for_workspace(int op, const Problem &pb, size_t ws_bytes)
{
    Plan pl = make_plan(op, pb);
    fit_two_parts(pl, ws_bytes);
    if (!(pl.sp || pl.win || (pl.lin && pl.fused_groups)) || ws_bytes >= pl.total) return pl;
    const Plan fp32 = make_plan(op, pb, false);
    return ws_bytes >= fp32.total ? fp32 : pl;
}

// ---------------------------------------------------------------------------
// Fully connected layers: x [N][I], w [O][I], y [N][O].  GEMM extents, operand
// orientation and the split of the reduction for fc_gemm_kernel (128 x 128
// tiles, 16 reduction elements per step).
// ---------------------------------------------------------------------------
struct FcPlan {
    int M, Nc, K;                 // output rows, output columns, reduction length
    int lda, ldb, ldd;
    bool at, bt;                  // operand A / B has its rows (columns) contiguous rather than k
    int mtiles, ntiles, ksplit, steps_per_split;
    size_t part_bytes;            // ksplit > 1: partial sums [ksplit][M][Nc], the whole workspace
    bool three_part;              // fc_split_kernel, else fc_gemm_kernel
};

inline int make_fc_plan(FcPlan &pl, int op, int N, int I, int O, int dtype)
{
    if (N <= 0 || I <= 0 || O <= 0) return kErrInvalidArg;
    if (op != kOpFwd && op != kOpBwdData && op != kOpBwdFilter) return kErrInvalidArg;
    if (I % 4 != 0 || O % 4 != 0) return kErrInvalidArg;      // 16-byte pieces along I and O
    if (dtype != kDtypeF32) return kErrBadDtype;
    const int64_t lim = (int64_t)1 << 31;
    if ((int64_t)N * I >= lim || (int64_t)N * O >= lim || (int64_t)O * I >= lim) return kErrTooLarge;
    if (op == kOpFwd) { pl.M = N; pl.Nc = O; pl.K = I; pl.lda = I; pl.ldb = I; pl.ldd = O; pl.at = false; pl.bt = false; }
    else if (op == kOpBwdData) { pl.M = N; pl.Nc = I; pl.K = O; pl.lda = O; pl.ldb = I; pl.ldd = I; pl.at = false; pl.bt = true; }
    else { pl.M = O; pl.Nc = I; pl.K = N; pl.lda = O; pl.ldb = I; pl.ldd = I; pl.at = true; pl.bt = true; }
    pl.mtiles = ceil_div(pl.M, 128);
    pl.ntiles = ceil_div(pl.Nc, 128);
    // aim at two work-groups per compute unit, with at least eight steps per range
    const int64_t tiles = (int64_t)pl.mtiles * pl.ntiles;
    const int steps = ceil_div(pl.K, kChunk);
    int ks = (int)std::min<int64_t>(std::max<int64_t>(1, 512 / tiles), std::max(1, steps / 8));
    ks = std::min(ks, 32);
    pl.steps_per_split = ceil_div(steps, ks);
    pl.ksplit = ceil_div(steps, pl.steps_per_split);
    pl.part_bytes = pl.ksplit > 1 ? (size_t)pl.ksplit * pl.M * pl.Nc * 4 : 0;
    if (tiles * pl.ksplit >= lim) return kErrTooLarge;
    // Three parts: 32-bit byte offsets, so tensors below 2^31 bytes; and reductions of two and more.  A sum of one product is
    // rounded once in fp32, while the six products leave out up to 2^-23 of it (2-norm error of 1024 x 768 such values 2.53e-8
    // against 2.60e-8; of two products 2.83e-8 against 2.61e-8, of sixteen 5.5e-8 against 2.9e-8).
    pl.three_part = pl.K > 1 && (int64_t)std::max(N, O) * I < lim / 4 && (int64_t)N * O < lim / 4;
    return kStatusOk;
}

}  // namespace convnet
#endif
