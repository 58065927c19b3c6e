"""fp32 passes on two half-precision parts, at the edges of their tiles and of the range of operands that they take, against the
CPU oracle.

Error bound, element by element, for a sum of L products.  An operand is h + l + e with |e| <= 2^-23 of it where it lies within
2^-28 of the tensor's largest, 2^-20 down to 2^-32; l l' <= 2^-22 is left out; the sum is rounded once per 16 products and split
range, and the 16 products of an instruction are aligned to the largest of them (2^-24 a product):
    |err| <= (L / 16 + 24) * 2^-24 * sum |x w|,     (L / 16 + 24 + 32) where there are operands below 2^-28
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


def within(got, ref, absref, length, more=0.0):
    bound = (length / 16.0 + 24.0 + more) * 2.0 ** -24 * absref
    err = np.abs(got.cpu().numpy().astype(np.float64) - ref)
    assert np.isfinite(err).all() and (err <= bound).all(), float((err / np.maximum(bound, 1e-300)).max())


class Pass:
    """One call of a pass and its oracle.  Operands a and w: input and filters, output gradient and filters, or (backward-filter)
    input and output gradient."""

    def __init__(self, op, shape):
        self.op, self.shape = op, shape
        N, C, H, W, K, R, st, pad = shape
        P, Q = hp.out_extent(H, R, st, pad), hp.out_extent(W, R, st, pad)
        x, w, y = (N, C, H, W), (K, C, R, R), (N, K, P, Q)
        self.a_shape, self.w_shape, self.out_shape = ((x, w, y), (y, w, x), (x, y, w))[op]
        self.length = (C * R * R, K * R * R, N * P * Q)[op]

    def operands(self, seed):
        return synth.gaussian(self.a_shape, seed), synth.gaussian(self.w_shape, seed + 1, 0.01 if self.op < 2 else 1.0)

    def gpu(self, a, w):
        _, _, H, W, _, R, st, pad = self.shape
        out = nan_like(self.out_shape)
        return (hp.conv_fwd(a, w, st, pad, y=out) if self.op == 0 else hp.conv_bwd_data(a, w, H, W, st, pad, dx=out)
                if self.op == 1 else hp.conv_bwd_filter(a, w, R, R, st, pad, dw=out))

    def three(self, a, w, route):
        """The same on three parts: in a workspace without room for what the operands' range is found with."""
        N, C, H, W, K, R, st, pad = self.shape
        less = route(self.op, *self.shape).workspace - 256
        small = route(self.op, *self.shape, workspace=less)
        assert small.kernels == "split" and not small.two_part
        buf, out = torch.empty(less, dtype=torch.uint8, device="cuda"), nan_like(self.out_shape)
        call = getattr(hp.lib(), ("conv_fwd", "conv_bwd_data", "conv_bwd_filter")[self.op])
        assert call(a.data_ptr(), w.data_ptr(), out.data_ptr(), N, C, H, W, K, R, R, st, pad, hp.DTYPE_F32, buf.data_ptr(), less,
                    torch.cuda.current_stream().cuda_stream) == hp.OK
        return out

    def ref(self, a, w):
        _, _, H, W, _, R, st, pad = self.shape
        return (oracle.conv_fwd(a, w, st, pad) if self.op == 0 else oracle.conv_bwd_data(a, w, H, W, st, pad) if self.op == 1
                else oracle.conv_bwd_filter(a, w, R, R, st, pad))

    def check(self, a, w, more=0.0):
        got = self.gpu(dev(a), dev(w))
        within(got, self.ref(a, w), self.ref(np.abs(a), np.abs(w)), self.length, more)
        return got


# Every tile; splits with an odd, an even and a shorter last range; channels that are no multiple of 16; samples of no multiple of
# four elements; strided passes whose classes have different counts of steps
SHAPES = [
    (0, (28, 512, 37, 50, 17, 7, 1, 3)),
    (0, (20, 368, 6, 16, 34, 5, 1, 2)),
    (0, (2, 384, 7, 15, 94, 5, 1, 2)),
    (0, (40, 256, 13, 13, 256, 3, 1, 1)),
    (0, (80, 114, 7, 39, 208, 3, 1, 1)),
    (0, (128, 256, 13, 13, 384, 3, 1, 1)),
    (1, (2, 16, 43, 29, 368, 7, 1, 3)),
    (1, (4, 223, 10, 36, 368, 5, 1, 2)),
    (1, (9, 94, 50, 44, 134, 5, 1, 2)),
    (1, (1, 368, 18, 31, 336, 5, 1, 2)),
    (1, (53, 100, 50, 36, 352, 7, 3, 3)),
    (1, (145, 222, 31, 7, 161, 7, 2, 3)),
]
WGRAD_SHAPES = [
    (2, (21, 176, 17, 48, 16, 7, 1, 3)),
    (2, (21, 176, 17, 48, 13, 7, 1, 3)),
    (2, (52, 176, 23, 40, 48, 7, 1, 3)),
    (2, (54, 175, 35, 31, 48, 5, 1, 2)),
    (2, (23, 512, 11, 24, 176, 5, 1, 2)),
    (2, (10, 512, 13, 19, 141, 5, 1, 2)),
    (2, (83, 128, 9, 48, 336, 3, 1, 1)),
    (2, (139, 224, 32, 15, 99, 2, 1, 1)),
]
SMALL = (0, (40, 256, 13, 13, 256, 3, 1, 1)), (1, (40, 256, 13, 13, 256, 3, 1, 1)), (2, (21, 176, 17, 48, 13, 7, 1, 3))


def test_these_shapes_take_every_tile(route):
    assert all(route(op, *shape).two_part for op, shape in (*SHAPES, *WGRAD_SHAPES, *SMALL))
    tiles = {(r.rows, r.columns) for op, shape in SHAPES for r in [route(op, *shape)]}
    assert tiles == {(128, 256), (128, 192), (128, 128), (96, 256), (64, 256), (32, 512)}
    tiles = {(route(op, *s).rows, s[1] % 16 != 0 or s[4] % 16 != 0) for op, s in WGRAD_SHAPES}
    assert tiles == {(rows, ragged) for rows in (32, 64, 96, 128) for ragged in (False, True)}


@pytest.mark.parametrize("op,shape", SHAPES + WGRAD_SHAPES)
def test_two_parts_stay_within_the_error_bound(op, shape, route):
    p = Pass(op, shape)
    a, w = p.operands(1001)
    two = p.check(a, w)
    assert not torch.equal(two, p.three(dev(a), dev(w), route))


# Dense operands, the output of a ReLU or of pooling for input, gradients with such layers' zeros: two parts (in two to eight
# segments) are no further from 64 bits than three, or three parts compute (None: either)
@pytest.mark.parametrize("op,shape", [(0, (40, 256, 13, 13, 256, 3, 1, 1)), (0, (128, 256, 13, 13, 384, 3, 1, 1)),
                                      (1, (64, 96, 13, 13, 256, 5, 1, 2)), (2, (21, 176, 17, 48, 16, 7, 1, 3)), (2, (120, 32, 40, 41, 256, 3, 1, 1)),
                                      (1, (40, 96, 17, 17, 256, 5, 1, 0))])
@pytest.mark.parametrize("kept_a,kept_w,sign,two", [(1.0, 1.0, False, True), (0.5, 1.0, False, None), (0.5, 1.0, True, None),
                                                    (0.9, 1.0, True, None), (0.5, 0.5, True, None), (0.02, 1.0, False, False)])
def test_two_parts_are_no_further_from_64_bits_than_three(op, shape, kept_a, kept_w, sign, two, route):
    p = Pass(op, shape)
    assert route(op, *shape).two_part
    a, w = p.operands(1011)
    rng = np.random.default_rng(3)
    if sign:
        a = np.abs(a)
    a, w = a * (rng.random(a.shape) < kept_a), w * (rng.random(w.shape) < kept_w)
    a, w = a.astype(np.float32), w.astype(np.float32)
    ad, wd = dev(a), dev(w)
    got, three = p.gpu(ad, wd), p.three(ad, wd, route)
    if op == 0 and sign:
        two = False                                        # a forward pass of a one-signed input
    assert two is None or torch.equal(got, three) != two
    ref = torch.from_numpy(p.ref(a, w)).cuda()
    err = [float((t.double() - ref).norm() / ref.norm()) for t in (got, three)]
    assert err[0] <= err[1]


# Tensors of other magnitudes: where two parts would be the further from 64 bits, three compute
def one_binade(s, rng):
    return rng.uniform(0.5, 1.0, s) * rng.choice([-1.0, 1.0], s)


def two_binades(s, rng):
    return rng.uniform(0.25, 1.0, s) * rng.choice([-1.0, 1.0], s)


def mostly_one_binade(s, rng):
    return np.where(rng.random(s) < 0.02, 0.01 * rng.standard_normal(s), one_binade(s, rng))


def signs(s, rng):
    return rng.choice([-1.0, 1.0], s)


def whole_numbers(s, rng):
    return rng.integers(-127, 128, s)


def off_centre(s, rng):
    return rng.standard_normal(s) + 3.0


def normal(s, rng):
    return rng.standard_normal(s)


def laplace(s, rng):
    return rng.laplace(size=s)


def heavy_tail(s, rng):
    return np.exp(2.0 * rng.standard_normal(s)) * rng.choice([-1.0, 1.0], s)


def below_one_outlier(s, rng):
    t = rng.uniform(0.5, 2.0, s) * rng.choice([-1.0, 1.0], s) * 2.0 ** -29
    t.flat[777] = 1.0
    return t


def below_many_outliers(s, rng):
    return rng.standard_normal(s) * np.where(rng.random(s) < 0.01, 1.0, 2.0 ** -28)


def samples_of_many_scales(s, rng):
    return rng.standard_normal(s) * 2.0 ** -(26.0 * rng.random((s[0],) + (1,) * (len(s) - 1)))


@pytest.mark.parametrize("op,shape", [*SMALL, (0, (32, 96, 28, 28, 128, 3, 1, 1))])
@pytest.mark.parametrize("draw_a,draw_w", [(normal, heavy_tail)] + [(d, d) for d in (one_binade, two_binades, mostly_one_binade, whole_numbers, off_centre, laplace,
                                                            below_one_outlier, below_many_outliers, samples_of_many_scales)] +
                         [(d, normal) for d in (one_binade, signs, whole_numbers, off_centre, below_one_outlier, samples_of_many_scales)] +
                         [(normal, d) for d in (one_binade, signs, whole_numbers, off_centre, below_one_outlier)])
def test_other_magnitudes_are_no_further_from_64_bits_than_three(op, shape, draw_a, draw_w, route):
    p = Pass(op, shape)
    assert route(op, *shape).two_part
    rng = np.random.default_rng(9)
    a, w = draw_a(p.a_shape, rng).astype(np.float32), draw_w(p.w_shape, rng).astype(np.float32)
    got, three = p.gpu(dev(a), dev(w)), p.three(dev(a), dev(w), route)
    assert draw_a is not laplace or not torch.equal(got, three)
    ref = torch.from_numpy(p.ref(a, w)).cuda()
    err = [float((t.double() - ref).norm() / ref.norm()) for t in (got, three)]
    assert err[0] <= err[1]


# One operand down to the line (2^-31 of the largest, and so half-precision subnormals), on it, and below; one up to 2^7 above the
# mean, and above: there, and wherever a tensor's largest operand is too small, too large, infinite or NaN, three parts compute
@pytest.mark.parametrize("op,shape", SMALL)
@pytest.mark.parametrize("second", [False, True])
@pytest.mark.parametrize("low,high,two", [(1.0, 1.0, True), (2.0 ** -31, 1.9, True), (2.0 ** -33, 1.0, False), (1.0, 2.0 ** 41, False),
                                          (2.0 ** -23, 2.0 ** 6, True), (1.0, 2.0 ** 7, False), (1.0, 3e38, False), (1e-40, 1.0, False),
                                          (1.0, np.inf, False), (1.0, np.nan, False)])
def test_the_range_of_operands_decides(op, shape, second, low, high, two, route):
    p = Pass(op, shape)
    a, w = p.operands(1015)
    f = lambda t: (np.clip(np.abs(t) / t.std(), 2.0 ** -10, 1.9) * np.sign(t)).astype(np.float32)
    a, w = f(a), f(w)
    (w if second else a).reshape(-1)[[5, 777]] = low, high
    ad, wd = dev(a), dev(w)
    got, three = p.gpu(ad, wd), p.three(ad, wd, route)
    assert torch.equal(got.view(torch.int32), three.view(torch.int32)) == (not two)
    if two:
        within(got, p.ref(a, w), p.ref(np.abs(a), np.abs(w)), p.length)


@pytest.mark.parametrize("op,shape", SMALL)
@pytest.mark.parametrize("spread", [12, 27, 31, 34, 120])
def test_operands_of_many_magnitudes(op, shape, spread):
    # magnitudes spread evenly over so many binades below 1; and one 1.0
    p = Pass(op, shape)
    a, w = p.operands(1021)
    rng = np.random.default_rng(7)
    f = lambda t: (np.sign(t) * 2.0 ** -(spread * rng.random(t.shape))).astype(np.float32)
    a, w = f(a), f(w)
    a.flat[0] = w.flat[0] = 1.0
    p.check(a, w, 32.0)


@pytest.mark.parametrize("op,shape", SMALL)
@pytest.mark.parametrize("low", [27, 31])
def test_small_operands_beside_one_large_one(op, shape, low, route):
    # everything near the lower end of the range, except for one operand that meets zeros: three parts
    p = Pass(op, shape)
    a, w = p.operands(1031)
    f = lambda t: np.clip(np.abs(t) / t.std(), 0.5, 2.0) * np.sign(t)
    a, w = (f(a) * 2.0 ** -(low - 2)).astype(np.float32), f(w).astype(np.float32)
    if op < 2:
        a[:, 11] = 0.0
        (w if op == 0 else w.transpose(1, 0, 2, 3))[:, 11] = 0.0
    else:
        a[3], w[3] = 0.0, 0.0
    a[3, 11, 2, 2] = 1.0
    assert torch.equal(p.check(a, w), p.three(dev(a), dev(w), route))


@pytest.mark.parametrize("op,shape", SMALL)
@pytest.mark.parametrize("second", [False, True])
@pytest.mark.parametrize("what", ["zero", "one sign"])
def test_the_first_channels_do_not_decide_alone(op, shape, second, what, route):
    # the first rows of every sample (filter) are no picture of the tensor: dead channels, channels of one sign
    p = Pass(op, shape)
    a, w = p.operands(1045)
    t = w if second else a
    t[:, :6] = 0.0 if what == "zero" else np.abs(t[:, :6])
    assert not torch.equal(p.check(a, w), p.three(dev(a), dev(w), route))


@pytest.mark.parametrize("op,shape", SMALL)
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38])
def test_infinities_and_nan_come_out_as_fp32_gives_them(op, shape, value):
    p = Pass(op, shape)
    a, w = p.operands(1041)
    w = np.abs(w) + np.float32(0.5)
    a[0, 9, 3, 4] = value
    with np.errstate(all="ignore"):
        got, ref = p.gpu(dev(a), dev(w)).cpu().numpy(), p.ref(a, w).astype(np.float32)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])


@pytest.mark.parametrize("op,shape", SMALL)
def test_zeros_and_an_empty_range(op, shape):
    p = Pass(op, shape)
    a, w = p.operands(1051)
    z = np.zeros_like
    for u, v in ((z(a), w), (a, z(w)), (z(a), z(w))):
        assert not bool(p.gpu(dev(u), dev(v)).any())


def test_slices_columns_and_epilogues(route):
    """Channel slices, columns of a grouped layer and the layer's epilogues: the
    bits of dense, separate and plain calls."""
    N, C, H, W, K, R = 5, 320, 20, 21, 320, 5
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    draw = lambda *s: torch.randn(s, device="cuda", generator=gen).clamp(-1.9, 1.9)
    assert route(0, N, C, H, W, K, R, 1, 2).two_part
    wide, w = draw(N, C + 8, H, W), draw(K, C, R, R) * 0.1
    dense = wide[:, 4:4 + C].contiguous()
    y = hp.conv_fwd(dense, w, 1, 2)
    assert torch.equal(hp.conv_fwd(wide[:, 4:4 + C], w, 1, 2), y)
    bias = torch.randn(K, device="cuda", generator=gen)
    assert torch.equal(hp.conv_fwd_bias_relu(dense, w, bias, 1, 2), torch.relu(y + bias[:, None, None]))
    dy, act = draw(N, C, H, W), torch.relu(torch.randn(N, K, H, W, device="cuda", generator=gen))
    wb = draw(C, K, R, R) * 0.1
    assert route(1, N, K, H, W, C, R, 1, 2).two_part
    dx = hp.conv_bwd_data(dy, wb, H, W, 1, 2)
    assert torch.equal(hp.conv_bwd_data_relu(dy, wb, act, 1, 2), torch.where(act > 0, dx, torch.zeros_like(dx)))
    assert route(0, N, 2 * C, H, W, 2 * K, R, 1, 2, groups=2).two_part
    x2, w2 = draw(N, 2 * C, H, W), draw(2 * K, C, R, R) * 0.1
    y2 = hp.conv_fwd_grouped(x2, w2, 1, 2, 2)
    assert not torch.equal(y, Pass(0, (N, C, H, W, K, R, 1, 2)).three(dense, w, route))
    for g in range(2):
        assert torch.equal(y2[:, K * g:K * (g + 1)], hp.conv_fwd(x2[:, C * g:C * (g + 1)], w2[K * g:K * (g + 1)], 1, 2))


# Columns of different operands: each takes two parts or three, and the scale, that it takes in a call of its own.  Two columns; six,
# which a preparing work-group looks up as it needs them (8 x 8 planes of one channel block: three columns within 128 positions)
@pytest.mark.parametrize("op,N,C,H,K,R,pad,groups", [(0, 5, 640, 20, 640, 5, 2, 2), (1, 5, 640, 20, 640, 5, 2, 2), (0, 4096, 96, 8, 768, 7, 0, 6),
                                                     (0, 48, 1152, 20, 768, 3, 1, 6), (1, 48, 768, 20, 1152, 3, 1, 6)])
def test_columns_of_different_operands_give_the_bits_of_separate_calls(op, N, C, H, K, R, pad, groups, route):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    assert route(op, N, C, H, H, K, R, 1, pad, groups=groups).two_part
    P = H + 2 * pad - R + 1
    act = torch.randn((N, C, H, H) if op == 0 else (N, K, P, P), device="cuda", generator=gen)
    w = torch.randn((K, C // groups, R, R), device="cuda", generator=gen) * 0.1
    a_cols, w_cols = act.chunk(groups, 1), w.chunk(groups, 0)
    a_cols[1][0, 3, 2, 1] = 2.0 ** 30                          # further above the others than two parts hold
    if groups > 2:
        w_cols[2][1, 2, 0, 1] = float("inf")
        a_cols[4].mul_(2.0 ** 12)
        a_cols[5].abs_()
    one = lambda a, u: hp.conv_fwd(a, u, 1, pad) if op == 0 else hp.conv_bwd_data(a, u, H, H, 1, pad)
    got = hp.conv_fwd_grouped(act, w, 1, pad, groups) if op == 0 else hp.conv_bwd_data_grouped(act, w, H, H, 1, pad, groups)
    for g, y in enumerate(got.chunk(groups, 1)):
        want = one(a_cols[g].contiguous(), w_cols[g].contiguous())
        assert torch.equal(y.contiguous().view(torch.int32), want.view(torch.int32)), g


def test_a_column_does_not_change_the_backward_filter_of_another():
    N, C, H, K, R = 64, 96, 27, 256, 5
    gen = torch.Generator(device="cuda")
    gen.manual_seed(8)
    x, dy = (torch.randn(s, device="cuda", generator=gen) for s in ((N, C, H, H), (N, K, H, H)))
    dw = hp.conv_bwd_filter_grouped(x, dy, R, R, 1, 2, 2)
    x[0, 50, 3, 3], dy[0, 200, 2, 2] = float("inf"), 2.0 ** -40
    again = hp.conv_bwd_filter_grouped(x, dy, R, R, 1, 2, 2)
    assert torch.equal(again[:K // 2], dw[:K // 2]) and not torch.equal(again[K // 2:], dw[K // 2:])


def test_a_call_can_be_captured_and_follows_its_operands(route):
    """What the operands' range says is found by each call on the GPU: a replayed graph takes two parts or three as they are then."""
    p = Pass(*SMALL[0])
    a, w = (dev(t) for t in p.operands(1061))
    out, ws = nan_like(p.out_shape), hp.Workspace("cuda")
    st, pad = p.shape[6:]
    hp.conv_fwd(a, w, st, pad, y=out, ws=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        hp.conv_fwd(a, w, st, pad, y=out, ws=ws)
    small = a.clone()
    small[0, 0] *= 2.0 ** -40
    for data in (a.clone(), small, a * 1e-30, torch.relu(a), a.clone(), small):
        a.copy_(data)
        graph.replay()
        torch.cuda.synchronize()
        replayed = out.clone()
        assert torch.equal(replayed, hp.conv_fwd(a, w, st, pad, ws=hp.Workspace("cuda")))
