"""fp32 passes whose operands are split into three bfloat16 parts, at the edges of their tiles and of their value range,
against the CPU oracle.

Error bound, element by element, for a sum of L products: the products left out are at most 3 * 2^-24 of |x w| each, the
sum of the leading products is rounded once per 16 products and split range (2^-24 of a partial sum that |x| * |w| summed
bounds), and the 16 products of an instruction are aligned to the largest of them, at most 2^-24 of it lost per product:
    |err| <= (L / 16 + 24) * 2^-24 * sum |x w|
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1312_5853_amd import binding as hp
from paper_1312_5853_amd import synth

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def nan_like(shape):
    return torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")


def within(got, ref, absref, length):
    bound = (length / 16.0 + 24.0) * 2.0 ** -24 * absref
    err = np.abs(got.cpu().numpy().astype(np.float64) - ref)
    assert np.isfinite(err).all() and (err <= bound).all(), float((err / np.maximum(bound, 1e-300)).max())


# N, C, H, W, K, R, stride, pad, and which of forward (f) and backward-data (d) run on the three-part kernels: rows 1 above
# and at a tile height (32, 64, 96, 128), a column more and less than a tile (256, 512), channel counts that are no multiple
# of 16, one position, split reductions (few columns), an even filter, padding beyond half the filter, 224 rows (four tiles of
# 64, not seven of 32), each tile of the kernel
SHAPES = [
    ((16, 64, 16, 16, 128, 3, 1, 1), "f"),
    ((1, 128, 16, 17, 129, 3, 1, 1), "d"),
    ((7, 96, 13, 13, 97, 3, 1, 1), "fd"),
    ((3, 65, 15, 17, 64, 3, 1, 1), "f"),
    ((5, 64, 21, 21, 33, 3, 1, 1), "fd"),
    ((16, 64, 27, 27, 32, 5, 1, 2), "fd"),
    ((1, 1024, 1, 1, 1024, 1, 1, 0), "fd"),
    ((2, 384, 13, 13, 384, 3, 1, 1), "fd"),
    ((2, 112, 12, 10, 100, 4, 1, 3), "fd"),
    ((4, 100, 24, 19, 200, 7, 2, 3), "f"),
    ((6, 19, 25, 28, 229, 5, 1, 2), "fd"),
    ((28, 61, 29, 24, 384, 1, 1, 0), "f"),
    ((4, 70, 27, 27, 224, 3, 1, 1), "f"),
]


def test_these_shapes_take_every_tile_of_the_forward_kernel(route):
    tiles = {(r.rows, r.columns) for shape, passes in SHAPES for p in passes for r in [route("fd".index(p), *shape)]}
    assert tiles == {(128, 256), (128, 192), (128, 128), (96, 256), (64, 256), (32, 512)}


@pytest.mark.parametrize("shape,passes", SHAPES)
def test_split_passes_stay_within_the_error_bound(shape, passes, route):
    N, C, H, W, K, R, st, pad = shape
    assert all(route("fd".index(p), *shape).kernels == "split" for p in passes)
    P, Q = hp.out_extent(H, R, st, pad), hp.out_extent(W, R, st, pad)
    x, w, dy = synth.gaussian((N, C, H, W), 901), synth.gaussian((K, C, R, R), 902, 0.01), synth.gaussian((N, K, P, Q), 903)
    ax, aw, ady = np.abs(x), np.abs(w), np.abs(dy)
    xd, wd, dyd = dev(x), dev(w), dev(dy)
    if "f" in passes:
        y = hp.conv_fwd(xd, wd, st, pad, y=nan_like((N, K, P, Q)))
        within(y, oracle.conv_fwd(x, w, st, pad), oracle.conv_fwd(ax, aw, st, pad), C * R * R)
    if "d" in passes:
        dx = hp.conv_bwd_data(dyd, wd, H, W, st, pad, dx=nan_like((N, C, H, W)))
        within(dx, oracle.conv_bwd_data(dy, w, H, W, st, pad), oracle.conv_bwd_data(ady, aw, H, W, st, pad), K * R * R)


# More than two rounds of tiles: half as wide, two work-groups to a CU; each height, ragged last tiles, a strided pass, samples
# compared at both ends of the mini-batch
@pytest.mark.parametrize("op,shape", [
    (0, (192, 32, 33, 31, 128, 3, 1, 1)), (0, (150, 3, 127, 119, 96, 11, 4, 2)), (0, (133, 48, 33, 31, 60, 3, 1, 1)),
    (1, (133, 60, 33, 31, 48, 3, 1, 1)), (1, (131, 64, 33, 31, 40, 3, 2, 1)),
])
def test_split_passes_of_many_rounds_stay_within_the_error_bound(op, shape, route):
    N, C, H, W, K, R, st, pad = shape
    r = route(op, *shape)
    assert r.kernels == "split" and r.columns == 128
    P, Q = hp.out_extent(H, R, st, pad), hp.out_extent(W, R, st, pad)
    a = synth.gaussian((N, C, H, W) if op == 0 else (N, K, P, Q), 971)
    w = synth.gaussian((K, C, R, R), 972, 0.01)
    got = (hp.conv_fwd(dev(a), dev(w), st, pad, y=nan_like((N, K, P, Q))) if op == 0
           else hp.conv_bwd_data(dev(a), dev(w), H, W, st, pad, dx=nan_like((N, C, H, W))))
    assert bool(torch.isfinite(got).all())
    for part in (slice(0, 3), slice(N // 2, N // 2 + 3), slice(N - 3, N)):
        s = a[part]
        f = (lambda t, u: oracle.conv_fwd(t, u, st, pad)) if op == 0 else (lambda t, u: oracle.conv_bwd_data(t, u, H, W, st, pad))
        within(got[part], f(s, w), f(np.abs(s), np.abs(w)), (C if op == 0 else K) * R * R)


def same_pattern(got, ref):
    """Where the 64-bit result, as fp32, is infinite or NaN; the rest close to it."""
    g, r = got.cpu().numpy(), ref.astype(np.float32)
    assert np.array_equal(np.isnan(g), np.isnan(r)) and np.array_equal(np.isinf(g), np.isinf(r))
    assert np.array_equal(g[np.isinf(r)], r[np.isinf(r)])
    fin = np.isfinite(r)
    assert np.abs(g[fin].astype(np.float64) - ref[fin]).max() <= 1e-5 * max(np.abs(ref[fin]).max(), 1e-300)


# ... with the layer's epilogues in their stores, on channel slices of wider tensors, two columns together: the plain pass's bits;
# and special values, which a work-group of four waves computes again
def test_split_passes_of_many_rounds_with_epilogues_slices_and_columns(route):
    N, C, H, W, K, R, st, pad = shape = 192, 32, 33, 31, 128, 3, 1, 1
    assert route(0, *shape).columns == 128
    x, w = torch.randn(N, C + 8, H, W, device="cuda"), torch.randn(K, C, R, R, device="cuda") * 0.05
    dense = x[:, 4:4 + C].contiguous()
    y = hp.conv_fwd(dense, w, st, pad)
    wide = torch.full((N, K + 8, H, W), 7.0, device="cuda")
    hp.conv_fwd(x[:, 4:4 + C], w, st, pad, y=wide[:, 4:4 + K])
    assert torch.equal(wide[:, 4:4 + K], y) and bool((wide[:, :4] == 7.0).all()) and bool((wide[:, 4 + K:] == 7.0).all())
    bias = torch.randn(K, device="cuda")
    assert torch.equal(hp.conv_fwd_bias_relu(dense, w, bias, st, pad), torch.relu(y + bias[:, None, None]))
    back = 133, 60, 33, 31, 48, 3, 1, 1
    assert route(1, *back).columns == 128
    dy, wb = torch.randn(133, 48, 33, 31, device="cuda"), torch.randn(48, 60, 3, 3, device="cuda") * 0.05
    act = torch.relu(torch.randn(133, 60, 33, 31, device="cuda"))
    dx = hp.conv_bwd_data(dy, wb, 33, 31, 1, 1)
    assert torch.equal(hp.conv_bwd_data_relu(dy, wb, act, 1, 1), torch.where(act > 0, dx, torch.zeros_like(dx)))
    two = 128, 64, 33, 31, 256, 3, 1, 1
    assert route(0, *two, groups=2).columns == 128 and route(0, 128, 32, 33, 31, 128, 3, 1, 1).columns == 256
    x2, w2 = torch.randn(128, 64, 33, 31, device="cuda"), torch.randn(256, 32, 3, 3, device="cuda") * 0.05
    y2 = hp.conv_fwd_grouped(x2, w2, 1, 1, 2)
    for g in range(2):
        assert torch.equal(y2[:, 128 * g:128 * (g + 1)], hp.conv_fwd(x2[:, 32 * g:32 * (g + 1)], w2[128 * g:128 * (g + 1)], 1, 1))


STRIDE1 = 3, 96, 13, 13, 96, 3, 1, 1         # both passes on the three-part kernels


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38, -3.4e38])
def test_split_passes_give_infinities_and_nan_as_fp32_does(value, route):
    # one such value in a mini-batch: the windows that read it, and only they, show it.  It meets positive filters, so
    # that no infinity of the other sign and no zero arises beside it.
    assert route(0, *STRIDE1).kernels == route(1, *STRIDE1).kernels == "split"
    x, w = synth.gaussian((3, 96, 13, 13), 911), np.abs(synth.gaussian((96, 96, 3, 3), 912)) + np.float32(0.5)
    x[1, 37, 6, 12] = value
    with np.errstate(all="ignore"):
        same_pattern(hp.conv_fwd(dev(x), dev(w), 1, 1), oracle.conv_fwd(x, w, 1, 1))
        same_pattern(hp.conv_bwd_data(dev(x), dev(w), 13, 13, 1, 1), oracle.conv_bwd_data(x, w, 13, 13, 1, 1))


@pytest.mark.parametrize("value", [np.inf, np.nan, 3.4e38])
def test_split_passes_of_many_rounds_give_infinities_and_nan_as_fp32_does(value, route):
    shape = N, C, H, W, K, R, st, pad = 192, 32, 33, 31, 128, 3, 1, 1
    assert route(0, *shape).columns == 128
    x, w = synth.gaussian((N, C, H, W), 913), np.abs(synth.gaussian((K, C, R, R), 914)) + np.float32(0.5)
    x[101, 17, 16, 30] = value
    y = hp.conv_fwd(dev(x), dev(w), st, pad)
    with np.errstate(all="ignore"):
        same_pattern(y[99:104], oracle.conv_fwd(x[99:104], w, st, pad))
    assert bool(torch.isfinite(y[:99]).all()) and bool(torch.isfinite(y[104:]).all())


@pytest.mark.parametrize("scale", [1e-30, 1e-34, 1e-37])
def test_split_passes_keep_fp32_precision_for_tiny_values(scale, route):
    assert route(0, *STRIDE1).kernels == "split"
    x, w = synth.gaussian((3, 96, 13, 13), 921) * np.float32(scale), synth.gaussian((96, 96, 3, 3), 922)
    y, ref = hp.conv_fwd(dev(x), dev(w), 1, 1), oracle.conv_fwd(x, w, 1, 1)
    assert np.abs(y.cpu().numpy().astype(np.float64) - ref).max() <= 864 * 2.0 ** -24 * oracle.conv_fwd(np.abs(x), np.abs(w), 1, 1).max()


# Backward-filter: rows at and above the tile heights, filter and channel counts that are no multiple of 16, fewer than 32
# positions in a split's last step, strides 2 and 3 with windows that leave input rows unread, padding, an even filter,
# two row tiles, columns past the last block of a tile
WGRAD_SHAPES = [
    (28, 80, 16, 2, 128, 1, 2, 0),
    (59, 144, 2, 7, 64, 1, 2, 0),
    (64, 48, 13, 13, 96, 3, 1, 1),
    (8, 32, 13, 13, 32, 3, 1, 1),
    (6, 19, 25, 28, 229, 5, 1, 2),
    (3, 16, 16, 17, 129, 3, 1, 1),
    (5, 65, 15, 17, 64, 3, 1, 1),
    (9, 32, 31, 33, 33, 5, 1, 2),
    (24, 40, 31, 45, 72, 3, 2, 1),
    (16, 9, 64, 60, 24, 3, 2, 0),
    (6, 13, 40, 41, 40, 5, 3, 0),
    (36, 41, 8, 9, 28, 2, 1, 2),
    (33, 128, 13, 13, 144, 3, 1, 1),
    # partial sums of channel counts that are no multiple of four: 1, 2, 3, 4, 5 and 74 splits
    (2, 113, 6, 4, 56, 3, 1, 1),
    (9, 113, 6, 20, 187, 1, 2, 0),
    (6, 49, 16, 19, 105, 3, 2, 1),
    (10, 45, 18, 3, 94, 3, 1, 1),
    (2, 61, 19, 17, 106, 3, 1, 1),
    (28, 61, 30, 14, 356, 1, 1, 0),
]


def test_these_shapes_take_every_tile_of_the_backward_filter_kernel(route):
    # whole and ragged counts of channels and filters are kernels of their own
    tiles = {(route(2, *s).rows, s[1] % 16 != 0 or s[4] % 16 != 0) for s in WGRAD_SHAPES}
    assert tiles == {(rows, ragged) for rows in (32, 64, 96, 128) for ragged in (False, True)}


@pytest.mark.parametrize("shape", WGRAD_SHAPES)
def test_split_backward_filter_stays_within_the_error_bound(shape, route):
    N, C, H, W, K, R, st, pad = shape
    assert route(2, *shape).kernels == "split"
    P, Q = hp.out_extent(H, R, st, pad), hp.out_extent(W, R, st, pad)
    x, dy = synth.gaussian((N, C, H, W), 904), synth.gaussian((N, K, P, Q), 905)
    dw = hp.conv_bwd_filter(dev(x), dev(dy), R, R, st, pad, dw=nan_like((K, C, R, R)))
    within(dw, oracle.conv_bwd_filter(x, dy, R, R, st, pad),
           oracle.conv_bwd_filter(np.abs(x), np.abs(dy), R, R, st, pad), N * P * Q)


def test_split_backward_filter_of_two_columns_stays_within_the_error_bound(route):
    # (not the bits of the columns alone: the splits are chosen for the columns of a launch together, as the fp32 kernels do)
    N, C, K, R = 6, 96, 256, 5
    assert route(2, N, C, 27, 27, K, R, 1, 2, groups=2).kernels == "split"
    x, dy = synth.gaussian((N, C, 27, 27), 906), synth.gaussian((N, K, 27, 27), 907)
    dw = hp.conv_bwd_filter_grouped(dev(x), dev(dy), R, R, 1, 2, 2, dw=nan_like((K, C // 2, R, R)))
    for g in range(2):
        xs, ys = x[:, 48 * g:48 * g + 48], dy[:, 128 * g:128 * g + 128]
        within(dw[128 * g:128 * g + 128], oracle.conv_bwd_filter(xs, ys, R, R, 1, 2),
               oracle.conv_bwd_filter(np.abs(xs), np.abs(ys), R, R, 1, 2), N * 27 * 27)


WHOLE, RAGGED = (8, 32, 13, 13, 32, 3, 1, 1), (5, 65, 15, 17, 64, 3, 1, 1)


@pytest.mark.parametrize("shape", [WHOLE, RAGGED])
@pytest.mark.parametrize("value", [np.inf, np.nan, -3.4e38])
def test_split_backward_filter_gives_infinities_and_nan_as_fp32_does(value, shape, route):
    N, C, H, W, K, R, st, pad = shape
    assert route(2, *shape).kernels == "split"
    x, dy = synth.gaussian((N, C, H, W), 913), np.abs(synth.gaussian((N, K, H, W), 914)) + np.float32(0.5)
    x[1, 27, 6, W - 1] = value
    with np.errstate(all="ignore"):
        same_pattern(hp.conv_bwd_filter(dev(x), dev(dy), R, R, st, pad), oracle.conv_bwd_filter(x, dy, R, R, st, pad))


@pytest.mark.parametrize("shape", [WHOLE, RAGGED])
@pytest.mark.parametrize("scale", [1e-30, 1e-37])
def test_split_backward_filter_keeps_fp32_precision_for_tiny_values(scale, shape, route):
    N, C, H, W, K, R, st, pad = shape
    assert route(2, *shape).kernels == "split"
    x, dy = synth.gaussian((N, C, H, W), 922), synth.gaussian((N, K, H, W), 923) * np.float32(scale)
    dw, ref = hp.conv_bwd_filter(dev(x), dev(dy), R, R, st, pad), oracle.conv_bwd_filter(x, dy, R, R, st, pad)
    top = oracle.conv_bwd_filter(np.abs(x), np.abs(dy), R, R, st, pad).max()
    assert np.abs(dw.cpu().numpy().astype(np.float64) - ref).max() <= N * H * W * 2.0 ** -24 * top


# Few-channel stride-4 backward-filter with the input rows in LDS: one to four blocks of 16 positions, the last full, nearly
# full, half full and with one position; 104 and fewer quads of taps, an unused column in a quad; 49, 65 and 96 filters; odd padding;
# more (image, row range) units than work-groups; rows of the longest extent
ROW_SHAPES = [
    (86, 3, 40, 120, 96, 11, 4, 2),
    (300, 3, 51, 31, 50, 11, 4, 2),
    (128, 3, 30, 226, 96, 11, 4, 2),
    (131, 2, 33, 160, 65, 12, 4, 0),
    (154, 3, 24, 200, 49, 7, 4, 1),
    (77, 3, 43, 69, 96, 11, 4, 2),
    (259, 3, 27, 73, 96, 11, 4, 3),
]


@pytest.mark.parametrize("shape", ROW_SHAPES)
def test_split_row_kernel_stays_within_the_error_bound(shape, route):
    N, C, H, W, K, R, st, pad = shape
    P, Q = hp.out_extent(H, R, st, pad), hp.out_extent(W, R, st, pad)
    assert route(2, *shape).kernels == "split"
    x, dy = synth.gaussian((N, C, H, W), 951), synth.gaussian((N, K, P, Q), 952)
    dw = hp.conv_bwd_filter(dev(x), dev(dy), R, R, st, pad, dw=nan_like((K, C, R, R)))
    within(dw, oracle.conv_bwd_filter(x, dy, R, R, st, pad),
           oracle.conv_bwd_filter(np.abs(x), np.abs(dy), R, R, st, pad), N * P * Q)


# Special values in the input, in dy, and one of each in different places; Q = 29: column 200 lies under taps 0..8 of the
# last three positions and, of the columns that are staged, under no window of the positions past Q
@pytest.mark.parametrize("where", ["x", "dy", "both"])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38])
def test_split_row_kernel_gives_infinities_and_nan_as_fp32_does(value, where, route):
    shape = N, C, H, W, K, R, st, pad = 86, 3, 40, 120, 96, 11, 4, 2
    P, Q = hp.out_extent(H, R, st, pad), hp.out_extent(W, R, st, pad)
    assert route(2, *shape).kernels == "split"
    x, dy = np.abs(synth.gaussian((N, C, H, W), 953)) + np.float32(0.5), np.abs(synth.gaussian((N, K, P, Q), 954)) + np.float32(0.5)
    if where != "dy":
        x[1, 2, 17, W - 1] = value
    if where != "x":
        dy[2, 41, 3, 7] = np.nan if where == "both" else value
    with np.errstate(all="ignore"):
        same_pattern(hp.conv_bwd_filter(dev(x), dev(dy), R, R, st, pad), oracle.conv_bwd_filter(x, dy, R, R, st, pad))


# Output rows of four blocks of 16 positions: their reads reach past the staged columns.  Special values in early columns of rows
# that are staged while others are read, of rows behind a work-group's last, and on every call the same bits
@pytest.mark.parametrize("value", [np.nan, np.inf, 3.4e38, 2.0 ** 110])
def test_split_row_kernel_repeats_itself_where_a_staged_row_is_not_finite(value, route):
    shape = N, C, H, W, K, R, st, pad = 128, 3, 30, 226, 96, 11, 4, 2
    P, Q = hp.out_extent(H, R, st, pad), hp.out_extent(W, R, st, pad)
    assert route(2, *shape).kernels == "split" and Q == 55
    x, dy = synth.gaussian((N, C, H, W), 957), synth.gaussian((N, K, P, Q), 958)
    x[1, 0, 9, 0] = x[7, 1, 13, 11] = x[N - 1, 2, H - 1, 30] = value
    xd, dyd = dev(x), dev(dy)
    first = hp.conv_bwd_filter(xd, dyd, R, R, st, pad).view(torch.int32).clone()
    for _ in range(20):
        assert torch.equal(hp.conv_bwd_filter(xd, dyd, R, R, st, pad).view(torch.int32), first)
    with np.errstate(all="ignore"):
        g, ref = first.view(torch.float32).cpu().numpy(), oracle.conv_bwd_filter(x, dy, R, R, st, pad)
        r, ref_abs = ref.astype(np.float32), oracle.conv_bwd_filter(np.abs(x), np.abs(dy), R, R, st, pad)
    assert np.array_equal(np.isnan(g), np.isnan(r)) and np.array_equal(np.isinf(g), np.isinf(r))
    ok = np.isfinite(r)
    # in fp32 a product passes through the sum of its work-group's positions and that of the 256 work-groups, one rounding each
    bound = (N * P * Q / 256 + 256 + 24) * 2.0 ** -24 * ref_abs
    assert (np.abs(g[ok].astype(np.float64) - ref[ok]) <= bound[ok]).all()


def test_split_row_kernel_on_channel_slices(route):
    """Input and output gradient as channel slices of wider tensors: the bits of dense ones."""
    shape = N, C, H, W, K, R, st, pad = 86, 3, 40, 120, 96, 11, 4, 2
    P, Q = hp.out_extent(H, R, st, pad), hp.out_extent(W, R, st, pad)
    assert route(2, *shape).kernels == "split"
    x, dy = torch.randn(N, C + 5, H, W, device="cuda"), torch.randn(N, K + 8, P, Q, device="cuda")
    xs, dys = x[:, 4:4 + C], dy[:, 4:4 + K]
    x[:, :4], x[:, 4 + C:], dy[:, :4], dy[:, 4 + K:] = float("nan"), float("nan"), float("nan"), float("nan")
    got = hp.conv_bwd_filter(xs, dys, R, R, st, pad, dw=nan_like((K, C, R, R)))
    assert torch.equal(got, hp.conv_bwd_filter(xs.contiguous(), dys.contiguous(), R, R, st, pad))


# Every instance (one to four blocks of 16 positions) keeps its operands in registers: a call on shorter rows takes no longer than
# one on the longest (with spills in the loop rows of 47 took two to four times as long)
def test_split_row_kernel_takes_no_longer_on_shorter_rows(route):
    def time(W):
        shape = N, C, H, _, K, R, st, pad = 128, 3, 128, W, 96, 11, 4, 2
        assert route(2, *shape).kernels == "split"
        P, Q = hp.out_extent(H, R, st, pad), hp.out_extent(W, R, st, pad)
        x, dy = torch.randn(N, C, H, W, device="cuda"), torch.randn(N, K, P, Q, device="cuda")
        dw = torch.empty(K, C, R, R, device="cuda")
        best = float("inf")
        for _ in range(6):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            hp.conv_bwd_filter(x, dy, R, R, st, pad, dw=dw)
            start.record()
            for _ in range(10):
                hp.conv_bwd_filter(x, dy, R, R, st, pad, dw=dw)
            end.record()
            end.synchronize()
            best = min(best, start.elapsed_time(end))
        return best
    longest = time(224)
    for W in (192, 128, 64):
        assert time(W) <= 1.1 * longest, W


@pytest.mark.parametrize("scale", [1e-30, 1e-37])
def test_split_row_kernel_keeps_fp32_precision_for_tiny_values(scale, route):
    shape = N, C, H, W, K, R, st, pad = 86, 3, 40, 120, 96, 11, 4, 2
    P, Q = hp.out_extent(H, R, st, pad), hp.out_extent(W, R, st, pad)
    x, dy = synth.gaussian((N, C, H, W), 955), synth.gaussian((N, K, P, Q), 956) * np.float32(scale)
    dw, ref = hp.conv_bwd_filter(dev(x), dev(dy), R, R, st, pad), oracle.conv_bwd_filter(x, dy, R, R, st, pad)
    top = oracle.conv_bwd_filter(np.abs(x), np.abs(dy), R, R, st, pad).max()
    assert np.abs(dw.cpu().numpy().astype(np.float64) - ref).max() <= N * P * Q * 2.0 ** -24 * top


# Fully connected: a column or row more and less than a tile, reductions that end inside a step or a split range, one sample
@pytest.mark.parametrize("N,I,O", [(1, 36, 20), (5, 132, 124), (127, 260, 132), (129, 1000, 128), (33, 4100, 68)])
def test_split_fully_connected_stays_within_the_error_bound(N, I, O):
    x, w, dy = synth.gaussian((N, I), 931), synth.gaussian((O, I), 932, 0.01), synth.gaussian((N, O), 933)
    ax, aw, ady = np.abs(x), np.abs(w), np.abs(dy)
    within(hp.fc_fwd(dev(x), dev(w), y=nan_like((N, O))), oracle.fc_fwd(x, w), oracle.fc_fwd(ax, aw), I)
    within(hp.fc_bwd_data(dev(dy), dev(w), dx=nan_like((N, I))), oracle.fc_bwd_data(dy, w), oracle.fc_bwd_data(ady, aw), O)
    within(hp.fc_bwd_filter(dev(x), dev(dy), dw=nan_like((O, I))), oracle.fc_bwd_filter(x, dy),
           oracle.fc_bwd_filter(ax, ady), N)


@pytest.mark.parametrize("value", [np.inf, np.nan, -3.4e38])
def test_split_fully_connected_gives_infinities_and_nan_as_fp32_does(value):
    x, w = synth.gaussian((9, 260), 934), np.abs(synth.gaussian((132, 260), 935)) + np.float32(0.5)
    x[3, 259] = value
    with np.errstate(all="ignore"):
        same_pattern(hp.fc_fwd(dev(x), dev(w)), oracle.fc_fwd(x, w))
        wt = np.ascontiguousarray(w.T)                                      # a reduction over 260 outputs
        same_pattern(hp.fc_bwd_data(dev(x), dev(wt)), oracle.fc_bwd_data(x, wt))
        dy = np.abs(synth.gaussian((9, 132), 936)) + np.float32(0.5)
        same_pattern(hp.fc_bwd_filter(dev(x), dev(dy)), oracle.fc_bwd_filter(x, dy))


def test_split_fully_connected_keeps_fp32_precision_for_tiny_values():
    x, w = synth.gaussian((9, 260), 937) * np.float32(1e-36), synth.gaussian((132, 260), 938)
    y, ref = hp.fc_fwd(dev(x), dev(w)), oracle.fc_fwd(x, w)
    assert np.abs(y.cpu().numpy().astype(np.float64) - ref).max() <= 260 * 2.0 ** -24 * oracle.fc_fwd(np.abs(x), np.abs(w)).max()


# A sum of one product is that product rounded once, whichever way the extents would send it
def test_a_single_product_is_correctly_rounded(route):
    x, dy = synth.gaussian((1, 1000), 945), synth.gaussian((1, 252), 946)
    assert np.array_equal(hp.fc_bwd_filter(dev(x), dev(dy)).cpu().numpy(), dy.T * x)
    shape = 1, 397, 1, 1, 21, 1, 1, 0
    assert route(2, *shape).kernels != "split" and route(2, 2, *shape[1:]).kernels == "split"
    x, dy = synth.gaussian((1, 397, 1, 1), 947), synth.gaussian((1, 21, 1, 1), 948)
    dw = hp.conv_bwd_filter(dev(x), dev(dy), 1, 1, 1, 0).cpu().numpy()
    assert np.array_equal(dw.reshape(21, 397), dy.reshape(21, 1) * x.reshape(1, 397))


# Strided backward-data as stride-1 passes over the residue classes: one of each stride, extents that leave input rows
# unread, a filter smaller than the stride (classes without taps), padding of half a filter and more, odd channel counts
@pytest.mark.parametrize("shape", [
    (24, 40, 31, 45, 72, 3, 2, 1),
    (9, 24, 30, 31, 33, 3, 2, 1),
    (5, 17, 29, 28, 48, 5, 3, 2),
    (6, 65, 17, 19, 64, 2, 3, 0),
    (3, 130, 31, 33, 100, 7, 4, 3),
    (2, 48, 23, 25, 40, 3, 2, 3),
])
def test_split_strided_backward_data_stays_within_the_error_bound(shape, route):
    N, C, H, W, K, R, st, pad = shape
    assert route(1, *shape).kernels == "split"
    P, Q = hp.out_extent(H, R, st, pad), hp.out_extent(W, R, st, pad)
    w, dy = synth.gaussian((K, C, R, R), 941, 0.01), synth.gaussian((N, K, P, Q), 942)
    ref, refabs = oracle.conv_bwd_data(dy, w, H, W, st, pad), oracle.conv_bwd_data(np.abs(dy), np.abs(w), H, W, st, pad)
    within(hp.conv_bwd_data(dev(dy), dev(w), H, W, st, pad, dx=nan_like((N, C, H, W))), ref, refabs, K * R * R)
    act = synth.gaussian((N, C, H, W), 943)
    got = hp.conv_bwd_data_relu(dev(dy), dev(w), dev(act), st, pad, dx=nan_like((N, C, H, W)))
    within(got, np.where(act > 0, ref, 0.0), refabs, K * R * R)
    dy[0, 3, 1, 1] = np.inf                                  # positive filters: only the windows' positions show it
    with np.errstate(all="ignore"):
        aw = np.abs(w) + np.float32(0.5)
        same_pattern(hp.conv_bwd_data(dev(dy), dev(aw), H, W, st, pad), oracle.conv_bwd_data(dy, aw, H, W, st, pad))


# Few channels, stride > 1: the input positions under an output position become channels.  Strides 2, 3 and 4, filters that
# are no multiple of the stride, odd extents and padding (no pairs of columns), a split reduction, rows of two tiles
@pytest.mark.parametrize("shape", [
    (12, 3, 40, 44, 96, 11, 4, 2),
    (30, 3, 47, 51, 48, 11, 4, 1),
    (20, 8, 33, 36, 64, 7, 2, 3),
    (33, 20, 23, 22, 40, 7, 2, 3),
    (1, 9, 29, 27, 20, 10, 3, 1),
    (25, 2, 61, 64, 33, 8, 4, 4),
])
def test_split_folded_passes_stay_within_the_error_bound(shape, route):
    N, C, H, W, K, R, st, pad = shape
    assert route(0, *shape).fold == st
    P, Q = hp.out_extent(H, R, st, pad), hp.out_extent(W, R, st, pad)
    x, w = synth.gaussian((N, C, H, W), 961), synth.gaussian((K, C, R, R), 962, 0.01)
    dy, b = synth.gaussian((N, K, P, Q), 963), synth.gaussian((K,), 964)
    y, yabs = oracle.conv_fwd(x, w, st, pad), oracle.conv_fwd(np.abs(x), np.abs(w), st, pad)
    within(hp.conv_fwd(dev(x), dev(w), st, pad, y=nan_like((N, K, P, Q))), y, yabs, C * R * R)
    b4 = b.reshape(1, -1, 1, 1)
    within(hp.conv_fwd_bias_relu(dev(x), dev(w), dev(b), st, pad, y=nan_like((N, K, P, Q))), np.maximum(y + b4, 0.0),
           yabs + np.abs(b4), C * R * R)
    within(hp.conv_bwd_filter(dev(x), dev(dy), R, R, st, pad, dw=nan_like((K, C, R, R))),
           oracle.conv_bwd_filter(x, dy, R, R, st, pad), oracle.conv_bwd_filter(np.abs(x), np.abs(dy), R, R, st, pad), N * P * Q)
    x[N - 1, 1, 6, 7] = np.inf
    with np.errstate(all="ignore"):
        aw, ady = np.abs(w) + np.float32(0.5), np.abs(dy) + np.float32(0.5)
        same_pattern(hp.conv_fwd(dev(x), dev(aw), st, pad), oracle.conv_fwd(x, aw, st, pad))
        same_pattern(hp.conv_bwd_filter(dev(x), dev(ady), R, R, st, pad), oracle.conv_bwd_filter(x, ady, R, R, st, pad))


def test_split_passes_tell_nan_from_values_that_only_their_first_part_makes_infinite(route):
    # a NaN, and in the same sums a finite value above the largest bfloat16 beside a zero: the NaN shows where fp32 has it,
    # and the zero times the large value stays zero
    assert route(0, *STRIDE1).kernels == route(2, *WHOLE).kernels == "split"
    x, w = synth.gaussian((3, 96, 13, 13), 971), np.abs(synth.gaussian((96, 96, 3, 3), 972)) + np.float32(0.5)
    x[1, 5, 6, 7] = np.nan
    x[2, 9, 3, 3] = np.float32(3.4e38)
    w[:, 9] = 0.0
    dy = np.abs(synth.gaussian((8, 32, 13, 13), 973)) + np.float32(0.5)
    xb = synth.gaussian((8, 32, 13, 13), 974)
    xb[3, 2, 8, 8], xb[4, 7, 1, 1] = np.nan, np.float32(3.4e38)
    dy[4] = 0.0
    a, b = synth.gaussian((9, 260), 975), np.abs(synth.gaussian((132, 260), 976)) + np.float32(0.5)
    a[3, 7], a[4, 9] = np.nan, np.float32(-3.4e38)
    b[:, 9] = 0.0
    with np.errstate(all="ignore"):
        same_pattern(hp.conv_fwd(dev(x), dev(w), 1, 1), oracle.conv_fwd(x, w, 1, 1))
        same_pattern(hp.conv_bwd_filter(dev(xb), dev(dy), 3, 3, 1, 1), oracle.conv_bwd_filter(xb, dy, 3, 3, 1, 1))
        same_pattern(hp.fc_fwd(dev(a), dev(b)), oracle.fc_fwd(a, b))


def near_where_finite(got, ref, refabs, length):
    """NaN and infinities where the 64-bit result has them; elsewhere the error bound of a finite input."""
    g = got.cpu().numpy().astype(np.float64)
    assert np.array_equal(np.isnan(g), np.isnan(ref)) and np.array_equal(g[np.isinf(ref)], ref[np.isinf(ref)])
    fin = np.isfinite(ref)
    assert (np.abs(g - ref)[fin] <= ((length / 16.0 + 24.0) * 2.0 ** -24 * refabs)[fin]).all()


# A folded filter is padded to whole strides with zeros, under which real input lies: row 37 = 4 * 7 - 2 + 11 is under the
# padded row of output row 7 and inside the windows of rows 8 and 9 (and 15 likewise for columns).  In sample 2 output row 7
# ends the first tile of 256 positions, the true windows lie in the next; in sample 5 they share one.
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf, 3.4e38])
def test_folded_forward_keeps_nan_and_infinities_inside_their_windows(value, route):
    shape = N, C, H, W, K, R, st, pad = 12, 3, 40, 44, 96, 11, 4, 2
    r = route(0, *shape)
    assert r.kernels == "split" and r.fold == 4 and r.columns == 256 and 2 * 90 + 7 * 10 + 4 < 256 <= 2 * 90 + 8 * 10
    x, w = np.abs(synth.gaussian((N, C, H, W), 981)), np.abs(synth.gaussian((K, C, R, R), 982)) + np.float32(0.5)
    b = synth.gaussian((K,), 983)
    refabs = oracle.conv_fwd(x, w, st, pad)
    x[2, 1, 37, 15] = value
    x[5, 0, 9, 9] = value
    with np.errstate(all="ignore"):
        ref = oracle.conv_fwd(x, w, st, pad)
        ref = np.where(np.isinf(ref.astype(np.float32)), np.copysign(np.inf, ref), ref)
        refabs = np.where(np.isfinite(ref), np.maximum(refabs, np.abs(ref)), refabs)
        near_where_finite(hp.conv_fwd(dev(x), dev(w), st, pad, y=nan_like(ref.shape)), ref, refabs, C * R * R)
        rb = ref + b.reshape(1, -1, 1, 1)
        near_where_finite(hp.conv_fwd_bias_relu(dev(x), dev(w), dev(b), st, pad, y=nan_like(ref.shape)),
                          np.where(rb > 0, rb, 0.0), refabs + np.abs(b).reshape(1, -1, 1, 1), C * R * R)


# A caller that brings the workspace of the fp32 kernels, as sized before there were others, is served by them; nothing past it
# is written.  Dense, strided, folded and grouped calls.
@pytest.mark.parametrize("op,shape,groups", [
    (0, (3, 96, 13, 13, 96, 3, 1, 1), 1), (0, (12, 3, 40, 44, 96, 11, 4, 2), 1), (0, (4, 192, 13, 13, 256, 3, 1, 1), 2),
    (1, (3, 96, 13, 13, 96, 3, 1, 1), 1), (1, (6, 65, 17, 19, 64, 2, 3, 0), 1),
    (2, (2, 75, 19, 10, 204, 3, 3, 1), 1), (2, (7, 14, 53, 12, 63, 5, 1, 2), 1),
])
def test_a_workspace_of_the_fp32_kernels_size_is_accepted(op, shape, groups, route):
    N, C, H, W, K, R, st, pad = shape
    want = route(op, *shape, groups=groups)
    assert want.kernels == "split"
    sizes = [b for b in range(0, want.workspace, 256) if route(op, *shape, groups=groups, workspace=b).kernels == "fp32"]
    assert sizes, "the fp32 kernels need less here"
    P, Q = hp.out_extent(H, R, st, pad), hp.out_extent(W, R, st, pad)
    x, w, dy = (dev(synth.gaussian(s, 985 + i)) for i, s in enumerate([(N, C, H, W), (K, C // groups, R, R), (N, K, P, Q)]))
    a, b, out = ((x, w, nan_like(dy.shape)), (dy, w, nan_like(x.shape)), (x, dy, nan_like(w.shape)))[op]
    buf = torch.full((sizes[0] + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    name = ("conv_fwd", "conv_bwd_data", "conv_bwd_filter")[op] + ("_grouped" if groups > 1 else "")
    more = (groups,) if groups > 1 else ()
    call = lambda nbytes: getattr(hp.lib(), name)(a.data_ptr(), b.data_ptr(), out.data_ptr(), N, C, H, W, K, R, R, st, pad,
                                                  *more, hp.DTYPE_F32, buf.data_ptr(), nbytes,
                                                  torch.cuda.current_stream().cuda_stream)
    assert call(sizes[0] - 1) == hp.ERR_WORKSPACE
    assert call(sizes[0]) == hp.OK
    assert bool((buf[sizes[0]:] == 0x5A).all())
    ax, aw, ady = (t.cpu().numpy() for t in (x, w, dy))
    cut = lambda t, g, axis: np.ascontiguousarray(np.split(t, groups, axis)[g])
    length = (C // groups * R * R, K // groups * R * R, N * P * Q)[op]
    for g in range(groups):
        gx, gw, gdy = cut(ax, g, 1), cut(aw, g, 0), cut(ady, g, 1)
        one = lambda f: ((lambda: oracle.conv_fwd(f(gx), f(gw), st, pad)), (lambda: oracle.conv_bwd_data(f(gdy), f(gw), H, W, st, pad)),
                         (lambda: oracle.conv_bwd_filter(f(gx), f(gdy), R, R, st, pad)))[op]()
        ref, absref = one(lambda t: t), one(np.abs)
        err = np.abs(cut(out.cpu().numpy(), g, 0 if op == 2 else 1).astype(np.float64) - ref)
        assert (err <= (length + 8) * 2.0 ** -24 * absref).all()                     # an fp32 sum of that length


# ---------------------------------------------------------------------------------------------------------------
# Operands of every magnitude.  Pass: extents N, C, H, W, K, R, stride, pad (fully connected: N, I, O), the axis of each
# operand that does not run along the reduction.  Both operands are N(0, 1) before they are scaled.
# ---------------------------------------------------------------------------------------------------------------
PASSES = {
    "fwd": ((3, 96, 13, 13, 96, 3, 1, 1), 0, 0),
    "fwd_folded": ((12, 3, 40, 44, 96, 11, 4, 2), 0, 0),
    "bwd_data": ((3, 96, 13, 13, 96, 3, 1, 1), 0, 1),
    "bwd_data_strided": ((6, 65, 17, 19, 64, 2, 3, 0), 0, 1),
    "bwd_filter": ((8, 32, 13, 13, 32, 3, 1, 1), 1, 1),
    "bwd_filter_tail": ((5, 65, 15, 17, 64, 3, 1, 1), 1, 1),
    "fc_fwd": ((9, 260, 132), 0, 0),
    "fc_bwd_data": ((9, 132, 260), 0, 1),
    "fc_bwd_filter": ((70, 132, 124), 1, 1),
}


def pass_operands(name, route):
    """The two operands, and a function of them: (GPU result, 64-bit result, 64-bit sum of magnitudes, reduction length)."""
    shape = PASSES[name][0]
    if name.startswith("fc_"):
        N, I, O = shape
        a, b = {"fc_fwd": ((N, I), (O, I)), "fc_bwd_data": ((N, O), (O, I)), "fc_bwd_filter": ((N, I), (N, O))}[name]
        gpu, ref = getattr(hp, name), getattr(oracle, name)
        length = {"fc_fwd": I, "fc_bwd_data": O, "fc_bwd_filter": N}[name]
        more = ()
    else:
        N, C, H, W, K, R, st, pad = shape
        P, Q = hp.out_extent(H, R, st, pad), hp.out_extent(W, R, st, pad)
        x, w, dy = (N, C, H, W), (K, C, R, R), (N, K, P, Q)
        op = 0 if name.startswith("fwd") else 1 if name.startswith("bwd_data") else 2
        assert route(op, *shape).kernels == "split" and (route(op, *shape).fold > 1) == (name == "fwd_folded")
        (a, b), more = (((x, w), (st, pad)), ((dy, w), (H, W, st, pad)), ((x, dy), (R, R, st, pad)))[op]
        gpu, ref = ((hp.conv_fwd, oracle.conv_fwd), (hp.conv_bwd_data, oracle.conv_bwd_data),
                    (hp.conv_bwd_filter, oracle.conv_bwd_filter))[op]
        length = (C * R * R, K * R * R, N * P * Q)[op]

    def run(a, b):
        return gpu(dev(a), dev(b), *more), ref(a, b, *more), ref(np.abs(a), np.abs(b), *more), length
    return synth.gaussian(a, 991), synth.gaussian(b, 992), run


def along(t, axis, index):
    return tuple([slice(None)] * axis + [index] + [slice(None)] * (t.ndim - axis - 1))


def rescale(a, axis_a, b, axis_b, kind):
    f = np.float32
    if kind == "tiny x large":
        return a * f(1e-37), b * f(1e18)
    if kind == "large x tiny":
        return a * f(1e15), b * f(1e-36)
    if kind == "subnormal x large":
        return a * f(1e-40), b * f(1e14)
    if kind == "tiny beside ordinary":          # one sample, filter or channel, of both operands
        a[along(a, axis_a, 1)] *= f(1e-37)
        b[along(b, axis_b, 2)] *= f(1e-37)
        a[along(a, axis_a, 2)] *= f(1e30)       # times 1e-37: sums around 1e-7
        return a, b
    if kind == "overflow of the accumulators":  # sums of both signs beyond 2^80
        return a * f(1e20), b * f(1e8)
    if kind == "large beside ordinary":
        a[along(a, axis_a, 1)] *= f(1e34)
        return a, b
    if kind == "large x zero":
        keep = b[along(b, axis_b, 1)] * f(1e-3)
        b = np.zeros_like(b)
        b[along(b, axis_b, 1)] = keep
        return a * f(1e34), b
    raise ValueError(kind)


KINDS = ["tiny x large", "large x tiny", "subnormal x large", "tiny beside ordinary", "overflow of the accumulators",
         "large beside ordinary", "large x zero"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("name", sorted(PASSES))
def test_split_passes_keep_fp32_precision_at_every_magnitude(name, kind, route):
    a, b, run = pass_operands(name, route)
    a, b = rescale(a, PASSES[name][1], b, PASSES[name][2], kind)
    got, ref, absref, length = run(a, b)
    # results below 2^-126 are subnormal: one rounding of at most 2^-150 per split range and one of their sum, and the fp32
    # kernels' products on top of that (`length` of them)
    bound = (length / 16.0 + 24.0) * 2.0 ** -24 * absref + (length + 16) * 2.0 ** -150
    err = np.abs(got.cpu().numpy().astype(np.float64) - ref)
    worst = float((err / bound).max())
    assert worst <= 1.0


@pytest.mark.parametrize("name", sorted(PASSES))
def test_split_passes_show_nan_beside_overflowing_accumulators(name, route):
    # everything overflows the accumulators, in one place there is a NaN: it shows where fp32 has it and nowhere else
    a, b, run = pass_operands(name, route)
    a, b = a * np.float32(1e20), b * np.float32(1e8)
    a.reshape(-1)[a.size // 2 + 1] = np.nan
    with np.errstate(all="ignore"):
        got, ref, absref, length = run(a, b)
    got = got.cpu().numpy().astype(np.float64)
    nan_as_it_should, fin = np.array_equal(np.isnan(got), np.isnan(ref)), np.isfinite(ref)
    bound = (length / 16.0 + 24.0) * 2.0 ** -24 * absref
    assert nan_as_it_should and fin.any() and (np.abs(got - ref)[fin] <= bound[fin]).all()


def test_fully_connected_tensors_of_two_gib_run_on_the_fp32_kernel():
    # 4096 x 131072 weights are 2^31 bytes: past the 32-bit offsets of the three-part kernel, all three passes
    N, I, O = 3, 131072, 4096
    gen = torch.Generator(device="cuda")
    gen.manual_seed(949)
    draw = lambda *shape: torch.empty(shape, device="cuda").normal_(0.0, 1.0, generator=gen)
    x, w, dy, b = draw(N, I), draw(O, I), draw(N, O), draw(O)
    ws = hp.Workspace("cuda")
    y, dx, dw = hp.fc_fwd(x, w, b, ws=ws), hp.fc_bwd_data(dy, w, ws=ws), hp.fc_bwd_filter(x, dy, ws=ws)
    worst = lambda got, ref, absref, length: float(((got.double() - ref).abs() / ((length + 8) * 2.0 ** -24 * absref)).max())
    x64, dy64 = x.double(), dy.double()
    dx_ref, dx_abs = torch.zeros_like(x64), torch.zeros_like(x64)
    for o in range(0, O, 256):
        wc, dyc = w[o:o + 256].double(), dy64[:, o:o + 256]
        ref, absref = x64 @ wc.t() + b[o:o + 256].double(), x64.abs() @ wc.abs().t() + b[o:o + 256].double().abs()
        assert worst(y[:, o:o + 256], ref, absref, I) <= 1.0
        assert worst(dw[o:o + 256], dyc.t() @ x64, dyc.abs().t() @ x64.abs(), N) <= 1.0
        dx_ref += dyc @ wc
        dx_abs += dyc.abs() @ wc.abs()
    assert worst(dx, dx_ref, dx_abs, O) <= 1.0
