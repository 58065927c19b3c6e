"""bf16 forward and backward-data with a tile's input window in LDS, at the edges of tiles, windows and channel chunks, against
the CPU oracle.

Error bound, element by element, of the fp32 results of a sum of L products: the products of bf16 values are exact, an
instruction adds 16 of them to the sum with one rounding and aligns them to the largest, as in test_gpu_split.py:
    |err| <= (L / 16 + 24) * 2^-24 * sum |x w|
A bf16 result is the fp32 one, rounded once.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_1312_5853_amd import binding as hp
from paper_1312_5853_amd import synth

pytestmark = pytest.mark.gpu


def bf16(shape, seed, std=1.0):
    t = torch.from_numpy(synth.gaussian(shape, seed, std)).to(torch.bfloat16)
    return t, t.to(torch.float32).numpy()


def within(got, ref, absref, length):
    bound = (length / 16.0 + 24.0) * 2.0 ** -24 * absref
    err = np.abs(got.cpu().numpy().astype(np.float64) - ref)
    assert np.isfinite(err).all() and (err <= bound).all(), float((err / np.maximum(bound, 1e-300)).max())


# pass (0 forward, 1 backward-data), then N, C, H, W, K, R, pad: every instance of the kernel (tile, two and three channel blocks
# per step, one and more chunks, some padded with blocks of zeros), odd and even counts of taps, rows that fill no tile, tiles
# across several samples, samples of a few positions, padding from none to the whole filter; three where a tap past the last is
# read behind the window
SHAPES = [
    (0, 4, 32, 30, 5, 45, 4, 2), (0, 3, 64, 12, 15, 54, 3, 1), (0, 9, 48, 32, 30, 47, 4, 0), (0, 1, 80, 9, 34, 60, 3, 2),
    (0, 66, 64, 32, 27, 36, 4, 3), (0, 53, 48, 31, 34, 37, 7, 6), (0, 2, 32, 29, 10, 80, 3, 2), (0, 5, 64, 6, 18, 96, 3, 0),
    (0, 3, 48, 6, 25, 119, 4, 0), (0, 1, 80, 17, 4, 224, 3, 2), (0, 59, 32, 32, 27, 83, 5, 4), (0, 50, 64, 26, 22, 67, 3, 2),
    (0, 64, 48, 30, 21, 131, 3, 1),
    (1, 9, 48, 9, 10, 32, 4, 0), (1, 2, 48, 33, 14, 64, 3, 0), (1, 39, 64, 24, 8, 48, 4, 0), (1, 2, 64, 13, 17, 80, 3, 0),
    (1, 70, 48, 29, 34, 112, 3, 0), (1, 62, 80, 4, 4, 32, 3, 0), (1, 4, 80, 5, 24, 64, 3, 0), (1, 5, 112, 12, 6, 48, 3, 0),
    (1, 2, 112, 19, 7, 80, 3, 0), (1, 70, 80, 33, 29, 32, 3, 2), (1, 41, 80, 29, 28, 64, 3, 1), (1, 61, 160, 10, 28, 48, 7, 0),
    (0, 96, 32, 42, 39, 48, 5, 2), (0, 3, 80, 4, 20, 240, 3, 0), (1, 2, 448, 3, 22, 80, 3, 0), (1, 1, 272, 3, 45, 80, 3, 1),
]


def test_these_shapes_take_every_instance(route):
    routes = [route(op, N, C, H, W, K, R, 1, pad, dtype=1) for op, N, C, H, W, K, R, pad in SHAPES]
    assert {(r.rows, r.columns, r.blocks, r.chunks > 1) for r in routes} == {
        (rows, width, blocks, several) for rows, widths in ((64, (256, 384)), (128, (128, 192))) for width in widths
        for blocks in (2, 3) for several in (False, True)} - {(64, 384, 3, True), (128, 192, 3, True)}      # (these fit no LDS)


@pytest.mark.parametrize("op,N,C,H,W,K,R,pad", SHAPES)
def test_window_passes_stay_within_the_error_bound(op, N, C, H, W, K, R, pad, route):
    assert route(op, N, C, H, W, K, R, 1, pad, dtype=1).kernels == "window"
    P, Q = hp.out_extent(H, R, 1, pad), hp.out_extent(W, R, 1, pad)
    wb, w = bf16((K, C, R, R), 962, 0.01)
    if op == 0:
        xb, x = bf16((N, C, H, W), 961)
        y = torch.full((N, K, P, Q), float("nan"), device="cuda")
        hp.conv_fwd(xb.cuda(), wb.cuda(), 1, pad, y=y)
        within(y, oracle.conv_fwd(x, w, 1, pad), oracle.conv_fwd(np.abs(x), np.abs(w), 1, pad), C * R * R)
        half = hp.conv_fwd(xb.cuda(), wb.cuda(), 1, pad, y=torch.empty((N, K, P, Q), dtype=torch.bfloat16, device="cuda"))
        assert torch.equal(half, y.to(torch.bfloat16))
    else:
        dyb, dy = bf16((N, K, P, Q), 963)
        dx = torch.full((N, C, H, W), float("nan"), device="cuda")
        hp.conv_bwd_data(dyb.cuda(), wb.cuda(), H, W, 1, pad, dx=dx)
        within(dx, oracle.conv_bwd_data(dy, w, H, W, 1, pad),
               oracle.conv_bwd_data(np.abs(dy), np.abs(w), H, W, 1, pad), K * R * R)
        half = hp.conv_bwd_data(dyb.cuda(), wb.cuda(), H, W, 1, pad,
                                dx=torch.empty((N, C, H, W), dtype=torch.bfloat16, device="cuda"))
        assert torch.equal(half, dx.to(torch.bfloat16))


# Bias and ReLU of the forward pass and the ReLU mask of backward-data in the kernel's stores: tiles of 64 and 128 rows, rows that
# fill none, one and several chunks (whose rows two groups of waves finish), fp32 and bf16 outputs.  The sums are the plain
# pass's, so the results are too, bit for bit.
@pytest.mark.parametrize("op,N,C,H,W,K,R,pad", [s for s in SHAPES if s[1] * s[2] * s[5] < 120000])
def test_window_epilogues_are_those_of_the_plain_sums(op, N, C, H, W, K, R, pad, route):
    assert route(op, N, C, H, W, K, R, 1, pad, dtype=1).kernels == "window"
    P, Q = hp.out_extent(H, R, 1, pad), hp.out_extent(W, R, 1, pad)
    wb, w = bf16((K, C, R, R), 972, 0.01)
    if op == 0:
        xb, x = bf16((N, C, H, W), 971)
        bias = torch.from_numpy(synth.gaussian((K,), 974, 0.1)).cuda()
        y = hp.conv_fwd(xb.cuda(), wb.cuda(), 1, pad)
        within(y, oracle.conv_fwd(x, w, 1, pad), oracle.conv_fwd(np.abs(x), np.abs(w), 1, pad), C * R * R)
        for b, relu in ((bias, True), (None, True), (bias, False)):
            want = y if b is None else y + b[:, None, None]
            want = torch.relu(want) if relu else want
            for dtype in (torch.float32, torch.bfloat16):
                out = torch.full((N, K, P, Q), float("nan"), dtype=dtype, device="cuda")
                assert torch.equal(hp.conv_fwd_bias_relu(xb.cuda(), wb.cuda(), b, 1, pad, relu=relu, y=out), want.to(dtype))
    else:
        dyb, dy = bf16((N, K, P, Q), 973)
        dx = hp.conv_bwd_data(dyb.cuda(), wb.cuda(), H, W, 1, pad)
        within(dx, oracle.conv_bwd_data(dy, w, H, W, 1, pad),
               oracle.conv_bwd_data(np.abs(dy), np.abs(w), H, W, 1, pad), K * R * R)
        act = torch.relu(torch.from_numpy(synth.gaussian((N, C, H, W), 975))).cuda()
        for dtype in (torch.float32, torch.bfloat16):
            out = torch.full((N, C, H, W), float("nan"), dtype=dtype, device="cuda")
            got = hp.conv_bwd_data_relu(dyb.cuda(), wb.cuda(), act.to(dtype), 1, pad, dx=out)
            assert torch.equal(got, torch.where(act > 0, dx, torch.zeros_like(dx)).to(dtype))


# Two and three columns in one launch, and filters that are not square: 64 and 128 rows, filled and not, one and several chunks
@pytest.mark.parametrize("op,N,C,H,W,K,R,S,pad,groups", [
    (0, 11, 160, 4, 6, 96, 3, 3, 2, 2), (0, 3, 64, 15, 15, 96, 4, 4, 2, 2), (0, 5, 64, 14, 5, 222, 3, 3, 2, 2),
    (0, 4, 240, 8, 6, 255, 3, 3, 2, 3), (0, 21, 144, 6, 5, 99, 4, 3, 2, 3), (1, 13, 66, 7, 10, 96, 4, 3, 2, 2),
    (1, 1, 192, 25, 15, 240, 3, 3, 2, 3), (1, 2, 285, 25, 5, 144, 3, 5, 2, 3), (1, 2, 238, 20, 5, 160, 3, 3, 2, 2),
    (0, 6, 32, 10, 4, 64, 4, 5, 3, 1), (0, 4, 64, 8, 13, 71, 2, 5, 1, 1), (0, 14, 48, 5, 4, 64, 5, 3, 2, 1),
    (1, 1, 55, 19, 24, 48, 2, 7, 1, 1), (1, 2, 96, 8, 19, 64, 1, 9, 0, 1), (1, 3, 144, 6, 9, 48, 5, 3, 0, 1),
    (1, 1, 192, 1, 171, 80, 1, 9, 0, 1),
])
def test_window_columns_and_oblong_filters_stay_within_the_error_bound(op, N, C, H, W, K, R, S, pad, groups, route):
    assert route(op, N, C, H, W, K, R, 1, pad, groups=groups, dtype=1, S=S).kernels == "window"
    P, Q = hp.out_extent(H, R, 1, pad), hp.out_extent(W, S, 1, pad)
    Cg, Kg = C // groups, K // groups
    wb, w = bf16((K, Cg, R, S), 982, 0.01)
    columns = lambda f, a: np.concatenate([f(a[:, g * (a.shape[1] // groups):(g + 1) * (a.shape[1] // groups)], g)
                                           for g in range(groups)], axis=1)
    if op == 0:
        srcb, src = bf16((N, C, H, W), 981)
        ref = lambda a, v: columns(lambda s, g: oracle.conv_fwd(s, v[g * Kg:(g + 1) * Kg], 1, pad), a)
        call = lambda out: (hp.conv_fwd_grouped(srcb.cuda(), wb.cuda(), 1, pad, groups, y=out) if groups > 1
                            else hp.conv_fwd(srcb.cuda(), wb.cuda(), 1, pad, y=out))
        shape, length = (N, K, P, Q), Cg * R * S
    else:
        srcb, src = bf16((N, K, P, Q), 983)
        ref = lambda a, v: columns(lambda s, g: oracle.conv_bwd_data(s, v[g * Kg:(g + 1) * Kg], H, W, 1, pad), a)
        call = lambda out: (hp.conv_bwd_data_grouped(srcb.cuda(), wb.cuda(), H, W, 1, pad, groups, dx=out) if groups > 1
                            else hp.conv_bwd_data(srcb.cuda(), wb.cuda(), H, W, 1, pad, dx=out))
        shape, length = (N, C, H, W), Kg * R * S
    got = call(torch.full(shape, float("nan"), device="cuda"))
    within(got, ref(src, w), ref(np.abs(src), np.abs(w)), length)
    assert torch.equal(call(torch.empty(shape, dtype=torch.bfloat16, device="cuda")), got.to(torch.bfloat16))


# Channel slices of wider tensors, input and output: the bits of dense tensors, and nothing written beside the slice
@pytest.mark.parametrize("op,N,C,H,W,K,R,pad", [(0, 9, 48, 32, 30, 47, 4, 0), (0, 5, 64, 6, 18, 96, 3, 0),
                                                (1, 39, 64, 24, 8, 48, 4, 0), (1, 2, 64, 13, 17, 80, 3, 0)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_window_passes_on_channel_slices(op, N, C, H, W, K, R, pad, dtype, route):
    assert route(op, N, C, H, W, K, R, 1, pad, dtype=1).kernels == "window"
    P, Q = hp.out_extent(H, R, 1, pad), hp.out_extent(W, R, 1, pad)
    wd = bf16((K, C, R, R), 992, 0.01)[0].cuda()
    ci, co = (C, K) if op == 0 else (K, C)
    hi, wi, ho, wo = (H, W, P, Q) if op == 0 else (P, Q, H, W)
    src = bf16((N, ci + 24, hi, wi), 991)[0].cuda()
    wide = torch.full((N, co + 24, ho, wo), 7.0, dtype=dtype, device="cuda")
    a, out = src[:, 8:8 + ci], wide[:, 16:16 + co]
    if op == 0:
        hp.conv_fwd(a, wd, 1, pad, y=out)
        want = hp.conv_fwd(a.contiguous(), wd, 1, pad, y=torch.empty((N, co, ho, wo), dtype=dtype, device="cuda"))
    else:
        hp.conv_bwd_data(a, wd, H, W, 1, pad, dx=out)
        want = hp.conv_bwd_data(a.contiguous(), wd, H, W, 1, pad, dx=torch.empty((N, co, ho, wo), dtype=dtype, device="cuda"))
    assert torch.equal(out, want)
    assert bool((wide[:, :16] == 7.0).all()) and bool((wide[:, 16 + co:] == 7.0).all())


# The columns of a grouped bf16 backward-filter in one launch: filters that fill a 128-row tile and that do not, two and three
# columns, several split ranges of the reduction, odd extents
@pytest.mark.parametrize("N,C,H,W,K,R,groups", [(6, 96, 27, 27, 256, 5, 2), (8, 48, 19, 23, 120, 3, 3), (12, 48, 19, 23, 360, 3, 3),
                                                (20, 96, 13, 16, 300, 3, 3)])
def test_grouped_backward_filter_stays_within_the_error_bound(N, C, H, W, K, R, groups, route):
    r = route(2, N, C, H, W, K, R, 1, R // 2, groups=groups, dtype=1)
    assert r.together
    xb, x = bf16((N, C, H, W), 968)
    dyb, dy = bf16((N, K, H, W), 969)
    refs = [oracle.conv_bwd_filter_grouped(a, b, R, R, 1, R // 2, groups) for a, b in ((x, dy), (np.abs(x), np.abs(dy)))]
    dw = hp.conv_bwd_filter_grouped(xb.cuda(), dyb.cuda(), R, R, 1, R // 2, groups,
                                    dw=torch.full((K, C // groups, R, R), float("nan"), device="cuda"))
    within(dw, *refs, N * H * W)
    # what one column needs is enough for one after the other
    one = hp.workspace_bytes(hp.OP_BWD_FILTER, N, C // groups, H, W, K // groups, R, R, 1, R // 2, hp.DTYPE_BF16)
    assert one < r.workspace
    assert not route(2, N, C, H, W, K, R, 1, R // 2, groups=groups, dtype=1, workspace=one).together
    dw.fill_(float("nan"))
    buf = torch.full((one + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    xd, dyd = xb.cuda(), dyb.cuda()
    call = lambda n: hp.lib().conv_bwd_filter_grouped(xd.data_ptr(), dyd.data_ptr(), dw.data_ptr(), N, C, H, W, K, R, R, 1, R // 2,
                                                      groups, hp.DTYPE_BF16, buf.data_ptr(), n,
                                                      torch.cuda.current_stream().cuda_stream)
    assert call(one - 1) == hp.ERR_WORKSPACE
    assert call(one) == hp.OK
    assert bool((buf[one:] == 0x5A).all())
    within(dw, *refs, N * H * W)


# NaN and infinities show in the windows that read them and in no others, chunks padded with zeros included
@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("shape", [(0, 1, 80, 9, 34, 60, 3, 2), (0, 3, 48, 6, 25, 119, 4, 0), (1, 2, 64, 13, 17, 80, 3, 0)])
def test_window_passes_keep_nan_and_infinities_inside_their_windows(value, shape, route):
    op, N, C, H, W, K, R, pad = shape
    assert route(op, N, C, H, W, K, R, 1, pad, dtype=1).kernels == "window"
    P, Q = hp.out_extent(H, R, 1, pad), hp.out_extent(W, R, 1, pad)
    wb = torch.from_numpy(np.abs(synth.gaussian((K, C, R, R), 964)) + np.float32(0.5)).to(torch.bfloat16)
    src = torch.from_numpy(synth.gaussian((N, C, H, W) if op == 0 else (N, K, P, Q), 965)).to(torch.bfloat16)
    src[N - 1, 5, 3, src.shape[3] - 1] = value
    a, w = src.to(torch.float32).numpy(), wb.to(torch.float32).numpy()
    with np.errstate(all="ignore"):
        got = (hp.conv_fwd(src.cuda(), wb.cuda(), 1, pad) if op == 0 else hp.conv_bwd_data(src.cuda(), wb.cuda(), H, W, 1, pad))
        ref = oracle.conv_fwd(a, w, 1, pad) if op == 0 else oracle.conv_bwd_data(a, w, H, W, 1, pad)
    g = got.cpu().numpy()
    assert np.array_equal(np.isnan(g), np.isnan(ref)) and np.array_equal(np.isinf(g), np.isinf(ref))


def test_a_workspace_of_the_staged_kernels_size_is_accepted(route):
    shape = 62, 80, 4, 4, 32, 3, 1, 0
    want = route(1, *shape, dtype=1)
    assert want.kernels == "window"
    less = [b for b in range(0, want.workspace, 256) if route(1, *shape, dtype=1, workspace=b).kernels != "window"]
    assert less, "the staged kernel needs less here"
    N, C, H, W, K, R, st, pad = shape
    P, Q = hp.out_extent(H, R, st, pad), hp.out_extent(W, R, st, pad)
    dyb, dy = bf16((N, K, P, Q), 966)
    wb, w = bf16((K, C, R, R), 967, 0.01)
    dx = torch.full((N, C, H, W), float("nan"), device="cuda")
    buf = torch.full((less[0] + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    dyd, wd = dyb.cuda(), wb.cuda()
    call = lambda n: hp.lib().conv_bwd_data(dyd.data_ptr(), wd.data_ptr(), dx.data_ptr(), N, C, H, W, K, R, R, st, pad, 1,
                                            buf.data_ptr(), n, torch.cuda.current_stream().cuda_stream)
    assert call(less[0] - 1) == hp.ERR_WORKSPACE
    assert call(less[0]) == hp.OK
    assert bool((buf[less[0]:] == 0x5A).all())
    within(dx, oracle.conv_bwd_data(dy, w, H, W, st, pad),
           oracle.conv_bwd_data(np.abs(dy), np.abs(w), H, W, st, pad), K * R * R)
