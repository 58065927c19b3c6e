"""Small convolution passes on the vector units, at the edges of their work-groups, against the CPU oracle.

A sum of L products in fp32 is at most (L + 8) * 2^-24 of the sum of their magnitudes away from the exact one; a bfloat16
result is rounded once more: 8 significant bits, at most 2^-8 of itself."""
import numpy as np
import pytest
import torch

import oracle
from paper_1312_5853_amd import binding as hp
from paper_1312_5853_amd import synth

pytestmark = pytest.mark.gpu

# N, C, H, W, K, R, stride, pad: one position, one row, 64 and 65 positions, 4 and 5 rows, 16 and 17 filters, reductions shorter
# than the sixteen wavefronts, strides with classes that no tap meets, padding beyond half the filter
SHAPES = [
    (4, 3, 32, 32, 16, 5, 1, 2),
    (1, 1, 1, 1, 1, 1, 1, 0),
    (1, 4, 8, 8, 17, 3, 1, 1),
    (5, 5, 13, 1, 4, 1, 1, 0),
    (2, 5, 11, 14, 5, 3, 2, 1),
    (3, 7, 10, 9, 3, 2, 3, 2),
    (7, 2, 33, 31, 16, 7, 2, 3),
]


def dev(a, dtype):
    t = torch.from_numpy(np.ascontiguousarray(a)).cuda()
    return t.to(torch.bfloat16) if dtype == "bf16" else t


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_direct_passes_stay_within_the_error_bound(shape, dtype, route):
    N, C, H, W, K, R, st, pad = shape
    assert all(route(op, *shape, dtype=0 if dtype == "f32" else 1).kernels == "direct" for op in range(3))
    P, Q = hp.out_extent(H, R, st, pad), hp.out_extent(W, R, st, pad)
    x, w = synth.gaussian((N, C, H, W), 951), synth.gaussian((K, C, R, R), 952)
    dy, b = synth.gaussian((N, K, P, Q), 953), synth.gaussian((K,), 954)
    if dtype == "bf16":
        x, w, dy = oracle.bf16_round(x), oracle.bf16_round(w), oracle.bf16_round(dy)
    ax, aw, ady = np.abs(x), np.abs(w), np.abs(dy)
    xd, wd, dyd = dev(x, dtype), dev(w, dtype), dev(dy, dtype)

    def within(got, ref, absref, length, rounded):
        bound = (length + 8) * 2.0 ** -24 * absref + (2.0 ** -8 * np.abs(ref) * 1.01 if rounded else 0.0)
        err = np.abs(got.float().cpu().numpy().astype(np.float64) - ref)
        assert np.isfinite(err).all() and (err <= bound).all()

    bf = dtype == "bf16"
    y, yabs = oracle.conv_fwd(x, w, st, pad), oracle.conv_fwd(ax, aw, st, pad)
    out = lambda like: torch.full_like(like, float("nan"))
    within(hp.conv_fwd(xd, wd, st, pad, y=out(dyd)), y, yabs, C * R * R, bf)
    yb = np.maximum(y + b.reshape(1, -1, 1, 1), 0.0)
    within(hp.conv_fwd_bias_relu(xd, wd, dev(b, "f32"), st, pad, y=out(dyd)), yb, yabs + np.abs(b).reshape(1, -1, 1, 1),
           C * R * R, bf)
    dx, dxabs = oracle.conv_bwd_data(dy, w, H, W, st, pad), oracle.conv_bwd_data(ady, aw, H, W, st, pad)
    within(hp.conv_bwd_data(dyd, wd, H, W, st, pad, dx=out(xd)), dx, dxabs, K * R * R, bf)
    within(hp.conv_bwd_data_relu(dyd, wd, xd, st, pad, dx=out(xd)), np.where(x > 0, dx, 0.0), dxabs, K * R * R, bf)
    dw = torch.full((K, C, R, R), float("nan"), device="cuda")
    within(hp.conv_bwd_filter(xd, dyd, R, R, st, pad, dw=dw), oracle.conv_bwd_filter(x, dy, R, R, st, pad),
           oracle.conv_bwd_filter(ax, ady, R, R, st, pad), N * P * Q, False)


def test_direct_passes_of_two_columns_equal_the_columns_alone(route):
    assert all(route(op, 2, 32, 9, 9, 8, 3, 1, 1, groups=2).kernels == "direct" for op in range(3))
    x, w, dy = (torch.from_numpy(synth.gaussian(s, 955 + i)).cuda()
                for i, s in enumerate([(2, 32, 9, 9), (8, 16, 3, 3), (2, 8, 9, 9)]))
    part = lambda t, g: t.chunk(2, 1)[g].contiguous()
    y, dx = hp.conv_fwd_grouped(x, w, 1, 1, 2), hp.conv_bwd_data_grouped(dy, w, 9, 9, 1, 1, 2)
    dw = hp.conv_bwd_filter_grouped(x, dy, 3, 3, 1, 1, 2)
    for g in range(2):
        wg = w[4 * g:4 * g + 4].contiguous()
        assert torch.equal(part(y, g), hp.conv_fwd(part(x, g), wg, 1, 1))
        assert torch.equal(part(dx, g), hp.conv_bwd_data(part(dy, g), wg, 9, 9, 1, 1))
        assert torch.equal(dw[4 * g:4 * g + 4], hp.conv_bwd_filter(part(x, g), part(dy, g), 3, 3, 1, 1))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(4, 3, 32, 32, 16, 5, 1, 0), (2, 3, 9, 9, 17, 3, 1, 0), (1, 1, 11, 11, 2, 3, 1, 0)])
def test_direct_passes_give_an_infinite_filter_value_as_an_infinity(shape, dtype, route):
    # positive operands, one filter with one infinity, no padding: infinite wherever that value takes part, as long as no group
    # of lanes multiplies it by the zero of an element that is not its own
    N, C, H, W, K, R, st, pad = shape
    for op in (0, 1):
        assert route(op, *shape, dtype=0 if dtype == "f32" else 1).kernels == "direct"
    P = H - R + 1
    x, dy = np.abs(synth.gaussian((N, C, H, W), 958)) + np.float32(0.5), np.abs(synth.gaussian((N, K, P, P), 959)) + np.float32(0.5)
    w = np.abs(synth.gaussian((K, C, R, R), 960)) + np.float32(0.5)
    w[1, 0, R - 1, 1] = np.inf
    y = hp.conv_fwd(dev(x, dtype), dev(w, dtype), st, pad).float().cpu().numpy()
    filters = np.isinf(y).all(axis=(0, 2, 3))
    assert filters[1] and filters.sum() == 1 and np.isfinite(np.delete(y, 1, 1)).all()
    dx = hp.conv_bwd_data(dev(dy, dtype), dev(w, dtype), H, W, st, pad).float().cpu().numpy()
    inner = dx[:, :, R - 1:P, R - 1:P]                         # positions that every tap reaches
    assert np.isinf(inner[:, 0]).all() and np.isfinite(inner[:, 1:]).all()


def test_calls_take_whole_number_objects_and_read_them_anew():
    x, w, dy = (dev(synth.gaussian(s, 963 + i), "f32") for i, s in enumerate([(2, 3, 9, 9), (4, 3, 3, 3), (2, 4, 9, 9)]))
    st, pad, nine = torch.tensor(2), np.array(1), np.array(9)
    assert torch.equal(hp.conv_fwd(x, w, st, pad), hp.conv_fwd(x, w, 2, 1))
    st.fill_(1)
    assert torch.equal(hp.conv_fwd(x, w, st, pad), hp.conv_fwd(x, w, 1, 1))
    assert torch.equal(hp.conv_fwd_bias_relu(x, w, None, st, pad), hp.conv_fwd_bias_relu(x, w, None, 1, 1))
    assert torch.equal(hp.conv_bwd_data(dy, w, nine, nine, st, pad), hp.conv_bwd_data(dy, w, 9, 9, 1, 1))
    assert torch.equal(hp.conv_bwd_data_relu(dy, w, x, st, pad), hp.conv_bwd_data_relu(dy, w, x, 1, 1))
    three = np.array(3)
    assert torch.equal(hp.conv_bwd_filter(x, dy, three, three, st, pad), hp.conv_bwd_filter(x, dy, 3, 3, 1, 1))
    with pytest.raises(TypeError):
        hp.conv_fwd(x, w, 1.0, 1)
    x, w = dev(synth.gaussian((2, 4, 8, 8), 966), "f32"), dev(synth.gaussian((4, 2, 3, 3), 967), "f32")
    assert torch.equal(hp.conv_fwd_grouped(x, w, st, pad, 2), hp.conv_fwd_grouped(x, w, 1, 1, 2))
