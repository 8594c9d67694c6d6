"""Polyphase kernels on the matrix cores: parity with the float64 oracle at the
sizes where their tiling can go wrong, and non-finite inputs.

Shapes: widths around the 8-column tiles and the 4-column blocks (odd ones
read rows at any alignment), heights around the two-row pairs and the vertical
segments, planes of 1 to 5 stages whose grids end at 1 x 1, batches that do not
fill the last group of resident planes, planes in region tiles whose last tile
is partial. The tolerances are the operator's (1e-5 of the largest value in
float32, 2e-2 in 16 bits)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_10805_amd import binding
from tests._gpu import TOL, rel_err, setup, to_np

pytestmark = pytest.mark.gpu

FORWARD = [
    (1, 1, 9, 4, 5, 1, "f32"), (3, 2, 9, 9, 3, 1, "f32"), (5, 2, 16, 17, 5, 2, "f32"), (7, 3, 15, 8, 5, 2, "bf16"),
    (2, 2, 31, 33, 5, 3, "f16"), (3, 1, 57, 55, 5, 3, "f32"), (2, 2, 56, 56, 5, 5, "bf16"), (19, 2, 14, 14, 5, 3, "bf16"),
    (4, 2, 63, 95, 5, 3, "f32"), (2, 1, 65, 94, 3, 4, "bf16"), (6, 2, 12, 100, 3, 2, "f16"), (2, 2, 100, 10, 5, 2, "bf16"),
    (11, 3, 20, 20, 3, 5, "f16"), (2, 2, 28, 30, 5, 4, "bf16"), (2, 1, 129, 131, 5, 1, "f32"), (2, 2, 120, 160, 5, 3, "bf16"),
    (1, 2, 226, 225, 3, 2, "f32"), (2, 1, 97, 203, 5, 2, "f16"), (3, 2, 7, 7, 5, 1, "bf16"), (70, 1, 8, 8, 3, 1, "f16"),
    (9, 3, 5, 4, 5, 1, "bf16"), (65, 130, 8, 4, 5, 1, "bf16"),
]


@pytest.mark.parametrize("B,C,H,W,k,L,dtype", FORWARD)
def test_forward_and_dx(B, C, H, W, k, L, dtype):
    inp, dev = setup(B, C, H, W, k, L, dtype, seed=B + H + W)
    want = oracle.forward(inp.x, inp.base_w, inp.base_scale, inp.level_w, inp.level_scale)
    assert rel_err(to_np(dev.forward()), want) < TOL[dtype]
    dx = binding.backward_data(dev.dy, dev.bw, dev.bs, dev.lw, dev.ls)
    torch.cuda.synchronize()
    ref = oracle.backward(inp.x, inp.dy, inp.base_w, inp.base_scale, inp.level_w, inp.level_scale)
    assert rel_err(to_np(dx), ref["dx"]) < TOL[dtype]


def footprint(H, W, y, x, k, L):
    """Outputs that depend on pixel (y, x): those whose 2^L x 2^L block lies
    within k // 2 blocks of the pixel's (the coarsest level's window holds
    every finer one's, and the base kernel's)."""
    R, m = k // 2, np.zeros((H, W), bool)
    j, i = y >> L, x >> L
    m[max(0, (j - R) << L):(j + R + 1) << L, max(0, (i - R) << L):(i + R + 1) << L] = True
    return m


@pytest.mark.parametrize("B,C,H,W,k,L,dtype", [(3, 2, 56, 56, 5, 1, "f32"), (2, 2, 40, 41, 5, 2, "bf16"),
                                               (5, 2, 28, 28, 3, 3, "f16"), (2, 1, 130, 128, 5, 1, "bf16")])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_non_finite_pixels_reach_their_outputs_only(B, C, H, W, k, L, dtype, value):
    """A non-finite pixel makes exactly the outputs that depend on it
    non-finite; every other value is the one without it."""
    _, dev = setup(B, C, H, W, k, L, dtype, seed=7)
    spots = [(0, 0, H // 3, W // 2 + 1), (B - 1, C - 1, H - 1, 0)]
    clean = dev.x.clone()
    for b, c, y, x in spots:
        clean[b, c, y, x] = 0
    want = binding.forward(clean, dev.bw, dev.bs, dev.lw, dev.ls)
    for b, c, y, x in spots:
        dev.x[b, c, y, x] = value
    got = dev.forward()
    bad = np.zeros((B, C, H, W), bool)
    for b, c, y, x in spots:
        bad[b, c] |= footprint(H, W, y, x, k, L)
    assert np.array_equal(~torch.isfinite(got).cpu().numpy(), bad)
    keep = torch.from_numpy(~bad).to(got.device)
    assert torch.equal(got[keep], want[keep])


@pytest.mark.parametrize("B,C,H,W,k,L,dtype", [(4, 768, 56, 56, 5, 1, "f32"), (4, 768, 56, 56, 5, 3, "bf16"),
                                               (4, 768, 28, 60, 3, 2, "f16"), (6, 256, 130, 128, 5, 1, "bf16")])
def test_non_finite_planes_one_after_another(B, C, H, W, k, L, dtype):
    """A workgroup's wavefronts store one batch of planes while others load the
    next: with nothing but NaN in all of them, every output is NaN."""
    _, dev = setup(1, C, 8, 8, k, L, dtype, seed=5)
    x = torch.full((B, C, H, W), float("nan"), dtype=dev.x.dtype, device=dev.x.device)
    y = binding.forward(x, dev.bw, dev.bs, dev.lw, dev.ls)
    assert bool(torch.isnan(y).all())


@pytest.mark.parametrize("B,C,H,W,k,L,dtype", [(3, 2, 56, 56, 5, 1, "f32"), (2, 2, 56, 56, 5, 3, "f32"),
                                               (2, 2, 40, 41, 5, 2, "bf16"), (2, 2, 28, 28, 5, 5, "bf16"),
                                               (5, 2, 28, 28, 3, 3, "f16"), (2, 1, 130, 128, 5, 1, "f32")])
def test_lowest_values_reach_their_outputs_only(B, C, H, W, k, L, dtype):
    """Pixels of the type's lowest value (a mask's): finite outputs, those that
    depend on one as the oracle has them, the others the same bits as without."""
    inp, dev = setup(B, C, H, W, k, L, dtype, seed=11)
    clean, bad = dev.x.clone(), np.zeros((B, C, H, W), bool)
    for b, c, y, x in [(0, 0, H // 3, W // 2 + 1), (B - 1, C - 1, H - 1, 0)]:
        dev.x[b, c, y, x] = torch.finfo(dev.x.dtype).min
        clean[b, c, y, x] = 0
        bad[b, c] |= footprint(H, W, y, x, k, L)
    got = dev.forward()
    assert bool(torch.isfinite(got).all())
    want = binding.forward(clean, dev.bw, dev.bs, dev.lw, dev.ls)
    keep = torch.from_numpy(~bad).to(got.device)
    assert torch.equal(got[keep], want[keep])
    ref = oracle.forward(to_np(dev.x), inp.base_w, inp.base_scale, inp.level_w, inp.level_scale)
    assert rel_err(to_np(got), ref) < TOL[dtype]


GRADIENT = [
    (1, 1, 9, 4, 5, 1, "bf16"), (3, 2, 11, 9, 3, 1, "f16"), (5, 2, 16, 17, 5, 2, "bf16"), (34, 1, 14, 14, 5, 2, "bf16"),
    (2, 2, 31, 33, 5, 3, "f16"), (3, 1, 57, 55, 5, 3, "bf16"), (3, 2, 48, 48, 5, 5, "bf16"), (19, 2, 14, 14, 3, 3, "bf16"),
    (4, 2, 63, 95, 5, 3, "bf16"), (2, 1, 65, 94, 3, 4, "bf16"), (6, 2, 12, 100, 3, 2, "f16"), (2, 2, 100, 10, 5, 2, "bf16"),
    (11, 3, 20, 20, 3, 5, "f16"), (2, 2, 28, 30, 5, 4, "bf16"), (7, 2, 40, 10, 5, 3, "f16"), (2, 1, 129, 131, 5, 1, "bf16"),
    (1, 2, 226, 225, 3, 1, "f16"), (3, 2, 7, 7, 5, 1, "bf16"), (70, 1, 8, 8, 3, 1, "f16"), (9, 3, 5, 4, 5, 1, "bf16"),
    (65, 3, 8, 5, 3, 1, "bf16"),
]


@pytest.mark.parametrize("B,C,H,W,k,L,dtype", GRADIENT)
def test_kernel_gradients(B, C, H, W, k, L, dtype):
    """16-bit inputs, float32 sums: every kernel gradient (and the bias's) to
    float32 accuracy on planes whose levels run in one pass or have one level
    (no intermediate is rounded to the storage type)."""
    inp, dev = setup(B, C, H, W, k, L, dtype, seed=B + 3 * H + W)
    bias = torch.linspace(-0.5, 0.5, C, device=dev.x.device)
    out = binding.backward(dev.x, dev.dy, dev.bw, dev.bs, dev.lw, dev.ls, bias=bias, need_dbias=True)
    torch.cuda.synchronize()
    ref = oracle.backward(inp.x, inp.dy, inp.base_w, inp.base_scale, inp.level_w, inp.level_scale)
    assert rel_err(to_np(out[0]), ref["dx"]) < TOL[dtype]
    assert rel_err(to_np(out[1]), ref["d_base_w"]) < 1e-5
    sdy = np.asarray(inp.dy, np.float64).sum((0, 2, 3))
    assert rel_err(to_np(out[2]), ref["d_base_scale"] + to_np(bias) * sdy) < 1e-5
    assert rel_err(to_np(out[5]), np.asarray(inp.base_scale, np.float64) * sdy) < 1e-5
    for l in range(L):
        assert rel_err(to_np(out[3][l]), ref["d_level_w"][l]) < 1e-5
        assert rel_err(to_np(out[4][l]), ref["d_level_scale"][l]) < 1e-5


def test_kernel_gradients_bitwise_reproducible():
    _, dev = setup(5, 3, 33, 35, 5, 4, "bf16", seed=3)
    a, b = dev.backward(), dev.backward()
    for p, q in zip((a[1], a[2], *a[3], *a[4]), (b[1], b[2], *b[3], *b[4])):
        assert torch.equal(p, q)


@pytest.mark.parametrize("B,C,H,W,k,L", [(2, 2, 126, 128, 5, 3), (2, 1, 127, 125, 3, 2), (1, 2, 137, 126, 5, 3),
                                         (1, 1, 226, 110, 3, 4)])
def test_float32_planes_with_a_sub_problem(B, C, H, W, k, L):
    """float32 planes in region tiles on both sides of the rule by which the
    tiles run polyphase; the sub-problem below them, without a base path, does
    not. Forward and combined backward, the operator's float32 tolerance."""
    inp, dev = setup(B, C, H, W, k, L, "f32", seed=11)
    want = oracle.forward(inp.x, inp.base_w, inp.base_scale, inp.level_w, inp.level_scale)
    assert rel_err(to_np(dev.forward()), want) < TOL["f32"]
    dx, dbw, dbs, dlw, dls = binding.backward(dev.x, dev.dy, dev.bw, dev.bs, dev.lw, dev.ls)
    torch.cuda.synchronize()
    ref = oracle.backward(inp.x, inp.dy, inp.base_w, inp.base_scale, inp.level_w, inp.level_scale)
    for got, name in [(dx, "dx"), (dbw, "d_base_w"), (dbs, "d_base_scale")]:
        assert rel_err(to_np(got), ref[name]) < TOL["f32"], name
    for l in range(L):
        assert rel_err(to_np(dlw[l]), ref["d_level_w"][l]) < TOL["f32"]
        assert rel_err(to_np(dls[l]), ref["d_level_scale"][l]) < TOL["f32"]


def haar_bands(v):
    """[B, C, H, W] -> the four bands of one orthonormal level, [B, C, 4, h, w], zero-extended."""
    v = torch.nn.functional.pad(v, [0, v.shape[-1] % 2, 0, v.shape[-2] % 2])
    a, b, c, d = v[..., 0::2, 0::2], v[..., 0::2, 1::2], v[..., 1::2, 0::2], v[..., 1::2, 1::2]
    return torch.stack([a + b + c + d, a + b - c - d, a - b + c - d, a - b - c + d], 2) / 2


def tap_sums(dz, v, k):
    """sum of dz times v shifted by every tap, over [B, ..., h, w]: v is zero
    outside its grid, except on planes of at most 8 x 8, where those products
    are left out."""
    h, w, R = v.shape[-2], v.shape[-1], k // 2
    pad = torch.nn.functional.pad(v, [R] * 4)
    inside = torch.nn.functional.pad(torch.ones_like(v), [R] * 4) > 0
    out = torch.empty(*v.shape[1:-2], k, k, dtype=v.dtype, device=v.device)
    for p in range(k):
        for t in range(k):
            prod = dz * pad[..., p:p + h, t:t + w]
            if tap_sums.tiny:
                prod = torch.where(inside[..., p:p + h, t:t + w], prod, torch.zeros((), dtype=v.dtype))
            out[..., p, t] = prod.sum((0, -1, -2))
    return out


@pytest.mark.parametrize("B,C,H,W,k,L,dtype", [
    (3, 2, 57, 55, 5, 1, "bf16"), (2, 2, 57, 57, 5, 2, "bf16"), (2, 2, 56, 56, 5, 3, "f16"), (20, 3, 13, 19, 3, 1, "bf16"),
    (19, 2, 14, 14, 3, 3, "bf16"), (3, 2, 48, 48, 5, 5, "bf16"), (2, 1, 129, 131, 5, 1, "f16"), (3, 2, 7, 7, 5, 1, "bf16")])
@pytest.mark.parametrize("side", ["x", "dy"])
@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")])
def test_non_finite_values_reach_the_kernel_gradients_that_see_them_only(B, C, H, W, k, L, dtype, side, value):
    """A non-finite value in the last row and column, and two of them close to
    each other: infinities keep their sign, taps that pair with none of them
    keep their values, as the sums over the plane have it in 64 bits."""
    inp, dev = setup(B, C, H, W, k, L, dtype, seed=2)
    t = getattr(dev, side)
    t[B - 1, 0, H - 1, W - 1] = value
    t[0, C - 1, H // 2, W // 2] = value
    t[0, C - 1, H // 2, W // 2 - 1] = float("inf")
    out = dev.backward()
    torch.cuda.synchronize()
    tap_sums.tiny = H <= 8 and W <= 8
    f64 = lambda v: v.double().cpu()  # noqa: E731
    x, dy = f64(dev.x), f64(dev.dy)
    pairs = [(out[1], tap_sums(dy, x, k), f64(dev.bs).view(-1, 1, 1))]
    for l in range(L):
        bx, bd = haar_bands(x), haar_bands(dy)
        pairs.append((out[3][l], tap_sums(bd, bx, k).reshape(4 * C, k, k), f64(dev.ls[l]).view(-1, 1, 1)))
        x, dy = bx[:, :, 0], bd[:, :, 0]
    for got, sums, scale in pairs:
        got, want = f64(got), sums * scale
        assert torch.equal(torch.isfinite(got), torch.isfinite(want))
        assert torch.equal(torch.nan_to_num(got, 0, 1, -1)[~torch.isfinite(want)],
                           torch.nan_to_num(want, 0, 1, -1)[~torch.isfinite(want)])
        keep = torch.isfinite(want)
        if keep.any():
            assert rel_err(got[keep].numpy(), want[keep].numpy()) < 1e-5


def plain_forward(x, bw, bs, lw, ls):
    """The operator in 64 bits, step by step, with IEEE infinities and NaN."""
    def conv(v, w):
        h, wd, k = v.shape[-2], v.shape[-1], w.shape[-1]
        out = torch.zeros_like(v)
        for p in range(k):
            for t in range(k):
                y0, x0 = p - k // 2, t - k // 2
                ys, xs = slice(max(0, -y0), h - max(0, y0)), slice(max(0, -x0), wd - max(0, x0))
                yi, xi = slice(max(0, y0), h + min(0, y0)), slice(max(0, x0), wd + min(0, x0))
                if ys.start < ys.stop and xs.start < xs.stop:  # (the zeros around a plane meet finite kernels only)
                    out[..., ys, xs] += v[..., yi, xi] * w[..., p, t, None, None]
        return out

    bands, sizes, v = [], [], x
    for _ in lw:
        sizes.append(v.shape[-2:])
        bands.append(haar_bands(v))
        v = bands[-1][:, :, 0]
    r = None
    for b, w, s, (h, wd) in reversed(list(zip(bands, lw, ls, sizes))):
        z = conv(b, (w * s.view(-1, 1, 1)).view(x.shape[1], 4, *w.shape[-2:]))
        if r is not None:
            z[:, :, 0] += r
        ll, lh, hl, hh = z.unbind(2)
        out = z.new_empty(*z.shape[:2], 2 * z.shape[-2], 2 * z.shape[-1])
        out[..., 0::2, 0::2], out[..., 0::2, 1::2] = (ll + lh + hl + hh) / 2, (ll + lh - hl - hh) / 2
        out[..., 1::2, 0::2], out[..., 1::2, 1::2] = (ll - lh + hl - hh) / 2, (ll - lh - hl + hh) / 2
        r = out[..., :h, :wd]
    return conv(x, bw * bs.view(-1, 1, 1)) + r


@pytest.mark.parametrize("B,C,H,W,k,L,dtype", [
    (3, 2, 57, 55, 5, 1, "f32"), (2, 2, 48, 48, 5, 2, "f32"), (2, 2, 57, 57, 5, 2, "bf16"), (2, 2, 56, 56, 5, 3, "bf16"),
    (3, 2, 56, 56, 5, 2, "f16"), (20, 3, 13, 19, 3, 4, "bf16"), (2, 1, 130, 128, 5, 1, "bf16"), (2, 2, 120, 160, 3, 3, "f16"),
    (17, 390, 17, 14, 5, 2, "f16"), (11, 512, 15, 11, 5, 4, "f16"), (9, 390, 14, 25, 3, 5, "bf16"),
    (23, 768, 11, 15, 5, 2, "f32"), (15, 768, 24, 13, 5, 3, "f32")])
def test_infinities_keep_their_sign(B, C, H, W, k, L, dtype):
    """y and dx where a pixel is infinite, and two of opposite sign are close:
    +inf, -inf or NaN as the step-by-step operator has it. (Level kernels
    without negative taps: the infinity of some outputs then survives.)"""
    inp, dev = setup(B, C, H, W, k, L, dtype, seed=9)
    for w in dev.lw:
        w.abs_()
    inf = float("inf")
    few = sorted({0, C - 1})  # the channels with infinities
    f64 = lambda v: v[:, few].double().cpu()  # noqa: E731
    par = lambda v: v.double().cpu().view(C, -1, *v.shape[1:])[few].flatten(0, 1)  # noqa: E731
    params = par(dev.bw), par(dev.bs), [par(w) for w in dev.lw], [par(s) for s in dev.ls]
    rotated = params[0].flip(-1, -2), params[1], [w.flip(-1, -2) for w in params[2]], params[3]
    for t in (dev.x, dev.dy):
        t[0, 0, H // 3, W // 2], t[0, 0, H // 3 + 1, W // 2 + 3], t[B - 1, C - 1, H - 1, W - 1] = inf, -inf, -inf
    dx = binding.backward_data(dev.dy, dev.bw, dev.bs, dev.lw, dev.ls)
    infinite = 0
    for got, want in ((dev.forward(), plain_forward(f64(dev.x), *params)), (dx, plain_forward(f64(dev.dy), *rotated))):
        got, bad = f64(got), ~torch.isfinite(want)
        assert torch.equal(~torch.isfinite(got), bad)
        assert torch.equal(torch.nan_to_num(got, 0, 1, -1)[bad], torch.nan_to_num(want, 0, 1, -1)[bad])
        assert rel_err(got[~bad].numpy(), want[~bad].numpy()) < TOL[dtype]
        infinite += int(torch.isinf(want).sum())
    assert infinite > 0


@pytest.mark.parametrize("B,C,H,W,k,L,dtype", [(3, 3, 57, 55, 5, 1, "f32"), (2, 3, 56, 56, 5, 3, "bf16"),
                                               (3, 3, 56, 56, 3, 2, "bf16"), (3, 3, 40, 41, 5, 1, "f16"),
                                               (2, 3, 130, 128, 5, 1, "bf16"), (3, 3, 7, 7, 5, 1, "bf16")])
@pytest.mark.parametrize("value", [float("inf"), -float("inf"), float("nan")])
def test_non_finite_kernels(B, C, H, W, k, L, dtype, value):
    """One non-finite tap of the base kernel and of a level's band make their
    channels what the sums have, and leave the other one as it is. (The zeros
    around a plane make NaN of them, but on planes of at most 8 x 8.)"""
    inp, dev = setup(B, C, H, W, k, L, dtype, seed=4)
    want = dev.forward()
    dev.bw[0, 1, 2] = value
    dev.lw[L - 1][4 + 2, 0, 0] = value
    got = dev.forward()
    assert torch.equal(got[:, 2], want[:, 2])
    inside = torch.zeros(B, H, W, dtype=torch.bool, device=got.device)
    R = k // 2
    inside[:, max(R - 1, 0):, :W - max(2 - R, 0)] = True  # outputs whose tap (1, 2) meets a pixel
    x = torch.nn.functional.pad(dev.x[:, 0].float(), [R] * 4)[:, 1:1 + H, 2:2 + W]
    ref = torch.where(inside, x * value, torch.full_like(x, float("nan")))
    if H <= 8:
        ref = torch.where(inside, ref, want[:, 0].float())
        assert rel_err(to_np(got[:, 0][~inside]), to_np(want[:, 0][~inside])) < TOL[dtype]
    else:
        assert not bool(torch.isfinite(got[:, 1]).any())
    bad = ~torch.isfinite(ref)
    assert torch.equal(torch.isfinite(got[:, 0]), ~bad)
    assert torch.equal(torch.nan_to_num(got[:, 0].float(), 0, 1, -1)[bad], torch.nan_to_num(ref, 0, 1, -1)[bad])


@pytest.mark.parametrize("B,C,H,W,k,L", [(2, 4, 56, 56, 5, 1), (17, 390, 17, 14, 5, 2), (13, 390, 35, 9, 3, 2),
                                         (2, 4, 130, 128, 5, 1)])
def test_float16_kernels_keep_float32_accuracy(B, C, H, W, k, L):
    """Taps 2^-34 of the channel's largest, each alone on a pixel: the outputs
    are those of the float32 taps, to half a step of float16 and the bound of the
    split, 2^-50 of the largest tap (two float16 pieces: 2^-39)."""
    g = torch.Generator(device="cuda").manual_seed(1)
    bw = (1 + torch.rand(C, k, k, generator=g, device="cuda")) * 2.0 ** -34
    bw[:, k // 2, k // 2] = 1
    one = torch.ones(C, device="cuda")
    lw, ls = [torch.zeros(4 * C, k, k, device="cuda")] * L, [torch.ones(4 * C, device="cuda")] * L
    x = torch.zeros(B, C, H, W, dtype=torch.float16, device="cuda")
    x[:, :, H // 2, W // 2] = 60000
    y = binding.forward(x, bw, one, lw, ls).double()
    want = torch.nn.functional.conv2d(x.double(), bw.double()[:, None], padding=k // 2, groups=C)
    want[:, :, H // 2, W // 2] = 60000
    assert float((y - want).abs().max()) <= 2.0 ** -25 + 60000 * 2.0 ** -50


@pytest.mark.parametrize("B,C,H,W,k,L,dtype", [(64, 12, 56, 56, 5, 3, "bf16"), (64, 12, 48, 48, 5, 5, "bf16"),
                                               (96, 8, 28, 28, 3, 3, "f16")])
def test_kernel_gradients_of_deep_levels_have_no_bias(B, C, H, W, k, L, dtype):
    """Rounding errors of one direction would add up over the planes: every
    level's gradient to 1.5e-7 of its norm (independent errors of float32 sums
    measure 5e-8 to 8e-8 here, and 3e-7 to 5e-7 with the bias), its mean error
    over a band to half of that."""
    inp, dev = setup(B, C, H, W, k, L, dtype, seed=6)
    out = dev.backward()
    tap_sums.tiny = False
    x, dy = dev.x.double(), dev.dy.double()
    for l in range(L):
        x, dy = haar_bands(x), haar_bands(dy)
        want = tap_sums(dy, x, k).cpu()
        got = (out[3][l].double() / dev.ls[l].double().view(-1, 1, 1)).view(C, 4, k, k).cpu()
        assert float((got - want).norm() / want.norm()) < 1.5e-7
        assert float((got - want).mean((0, 2, 3)).abs().max() / want.pow(2).mean().sqrt()) < 7.5e-8
        x, dy = x[:, :, 0], dy[:, :, 0]


# (problem, batches of the forward, of the kernel gradients): planes of a batch,
# batches of a workgroup and planes in its last, partial one. tests/test_planner.py
# checks that the library still plans them so.
GROUPS = [
    ((34, 390, 15, 11, 3, 1, "bf16"), (12, 3, 10), (17, 2, 17)), ((9, 390, 42, 14, 3, 2, "bf16"), (5, 2, 4), (5, 2, 4)),
    ((11, 768, 11, 9, 3, 3, "bf16"), (6, 2, 5), (6, 2, 5)), ((20, 390, 17, 10, 3, 4, "f16"), (7, 3, 6), (7, 3, 6)),
    ((9, 390, 14, 25, 3, 5, "bf16"), (5, 2, 4), (5, 2, 4)), ((43, 390, 14, 10, 5, 1, "bf16"), (15, 3, 13), (22, 2, 21)),
    ((17, 390, 17, 14, 5, 2, "f16"), (10, 2, 7), (9, 2, 8)), ((29, 390, 13, 9, 5, 3, "bf16"), (8, 4, 5), (8, 4, 5)),
    ((11, 512, 15, 11, 5, 4, "f16"), (6, 2, 5), (6, 2, 5)), ((9, 390, 13, 28, 5, 5, "bf16"), (7, 2, 2), (5, 2, 4)),
    ((33, 390, 11, 9, 3, 1, "f32"), (17, 2, 16), None), ((7, 390, 62, 11, 3, 2, "f32"), (4, 2, 3), None),
    ((5, 390, 61, 9, 3, 3, "f32"), (3, 2, 2), None), ((19, 390, 19, 7, 5, 1, "f32"), (10, 2, 9), None),
    ((23, 768, 11, 15, 5, 2, "f32"), (8, 3, 7), None), ((15, 768, 24, 13, 5, 3, "f32"), (4, 4, 3), None),
]


@pytest.mark.parametrize("spec,forward,gradient", GROUPS)
def test_batches_of_planes(spec, forward, gradient):
    """Several planes to a batch, several batches to a workgroup, the last one
    partial: y, dx and the kernel gradients."""
    B, C, H, W, k, L, dtype = spec
    test_forward_and_dx(B, C, H, W, k, L, dtype)
    if gradient:
        test_kernel_gradients(B, C, H, W, k, L, dtype)


# float32 in region tiles: one level, and a carry from the coarser ones
REGIONS = [(1, 96, 115, 113, 5, 1, "f32"), (1, 103, 116, 113, 3, 1, "f32"), (2, 64, 97, 69, 5, 3, "f32"),
           (3, 64, 123, 59, 3, 3, "f32")]


@pytest.mark.parametrize("B,C,H,W,k,L,dtype", REGIONS)
def test_float32_region_tiles(B, C, H, W, k, L, dtype):
    test_forward_and_dx(B, C, H, W, k, L, dtype)
    test_extreme_pixels_of_deeper_stages(B, C, H, W, k, L, dtype)


# polyphase forwards (in region tiles the last) with more than one stage
STAGES = [(2, 2, 56, 56, 5, 3, "bf16"), (2, 2, 57, 57, 5, 2, "bf16"), (17, 390, 17, 14, 5, 2, "f16"),
          (11, 512, 15, 11, 5, 4, "f16"), (9, 390, 14, 25, 3, 5, "bf16"), (23, 768, 11, 15, 5, 2, "f32"),
          (15, 768, 24, 13, 5, 3, "f32"), (5, 390, 61, 9, 3, 3, "f32"), (2, 2, 120, 160, 5, 1, "f16")]


@pytest.mark.parametrize("B,C,H,W,k,L,dtype", STAGES)
def test_extreme_pixels_of_deeper_stages(B, C, H, W, k, L, dtype):
    """The two tests above on planes whose stages all run polyphase."""
    test_non_finite_pixels_reach_their_outputs_only(B, C, H, W, k, L, dtype, float("nan"))
    test_non_finite_pixels_reach_their_outputs_only(B, C, H, W, k, L, dtype, float("inf"))
    test_lowest_values_reach_their_outputs_only(B, C, H, W, k, L, dtype)
