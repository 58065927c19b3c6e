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


# pass (0 forward, 1 backward-data), then N, C, H, W, K, R, pad: every tile, two and three channel blocks per step, one and more
# chunks (some padded with blocks of zeros), odd and even counts of taps, rows that fill no tile, tiles across several samples,
# samples of a few positions, padding from none to the whole filter
SHAPES = [
    (0, 4, 32, 30, 5, 45, 4, 2), (0, 3, 64, 12, 15, 54, 3, 1), (0, 9, 48, 32, 30, 47, 4, 0), (0, 1, 80, 9, 34, 60, 3, 2),
    (0, 66, 64, 32, 27, 36, 4, 3), (0, 53, 48, 31, 34, 37, 7, 6), (0, 2, 32, 29, 10, 80, 3, 2), (0, 5, 64, 6, 18, 96, 3, 0),
    (0, 3, 48, 6, 25, 119, 4, 0), (0, 1, 80, 17, 4, 224, 3, 2), (0, 59, 32, 32, 27, 83, 5, 4), (0, 50, 64, 26, 22, 67, 3, 2),
    (0, 64, 48, 30, 21, 131, 3, 1),
    (1, 9, 48, 9, 10, 32, 4, 0), (1, 2, 48, 33, 14, 64, 3, 0), (1, 39, 64, 24, 8, 48, 4, 0), (1, 2, 64, 13, 17, 80, 3, 0),
    (1, 70, 48, 29, 34, 112, 3, 0), (1, 62, 80, 4, 4, 32, 3, 0), (1, 4, 80, 5, 24, 64, 3, 0), (1, 5, 112, 12, 6, 48, 3, 0),
    (1, 2, 112, 19, 7, 80, 3, 0), (1, 70, 80, 33, 29, 32, 3, 2), (1, 41, 80, 29, 28, 64, 3, 1), (1, 61, 160, 10, 28, 48, 7, 0),
]


def test_these_shapes_take_every_tile(route):
    tiles = {(r.rows, r.columns) for op, N, C, H, W, K, R, pad in SHAPES for r in [route(op, N, C, H, W, K, R, 1, pad, dtype=1)]}
    assert tiles == {(64, 256), (64, 384), (128, 128), (128, 192)}


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


# The columns of a grouped bf16 backward-filter in one launch: filters that fill no 128-row tile, three columns, one and many
# split ranges of the reduction, odd extents
@pytest.mark.parametrize("N,C,H,W,K,R,groups", [(6, 96, 27, 27, 256, 5, 2), (3, 48, 19, 23, 120, 3, 3), (40, 64, 13, 15, 320, 3, 2)])
def test_grouped_backward_filter_stays_within_the_error_bound(N, C, H, W, K, R, groups):
    xb, x = bf16((N, C, H, W), 968)
    dyb, dy = bf16((N, K, H, W), 969)
    dw = hp.conv_bwd_filter_grouped(xb.cuda(), dyb.cuda(), R, R, 1, R // 2, groups,
                                    dw=torch.full((K, C // groups, R, R), float("nan"), device="cuda"))
    within(dw, oracle.conv_bwd_filter_grouped(x, dy, R, R, 1, R // 2, groups),
           oracle.conv_bwd_filter_grouped(np.abs(x), np.abs(dy), R, R, 1, R // 2, groups), N * H * W)


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
