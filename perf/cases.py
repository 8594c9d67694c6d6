"""Performance cases of the fused WTConv operator.

The cases are what a program that uses this package has it do: forwards for
serving and training steps (forward, then backward with the gradients of x and
of every parameter), from one small call to large planes, through the public
entry points: `binding.forward`, the prepared `binding.Forward` and
`binding.Backward`, and the `WTConv2d` module under autograd. Shapes are the
ConvNeXt-T stages (56, 28, 14 and 7 pixels), the odd 63 x 95 plane, the 224 x
224 plane and the paper's layer sweep (128 x 128 to 256 x 256 planes at B = 8),
with kernel sizes 3, 5 and 7 and float32, bfloat16 and float16 activations.
"""
import math

import torch
import torch.nn.functional as F

from paper_2608_10805_amd import autograd, binding

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
DEVICE = "cuda"


def _case(name, task, api, B, C, H, W, k, L, dtype, bias=False):
    return {"name": name, "task": task, "api": api, "B": B, "C": C, "H": H, "W": W, "k": k, "L": L,
            "dtype": dtype, "bias": bias}


def listed():
    return [
        # one small call of an eager program: launch and host latency decide
        _case("infer_small_32", "infer", "call", 2, 16, 32, 32, 5, 1, "f32"),
        # serving the first ConvNeXt-T stage in float32, calls prepared once
        _case("infer_stage1_f32", "infer", "prepared", 64, 96, 56, 56, 5, 3, "f32"),
        # a high-resolution feature map in half precision, the paper's inference sweep
        _case("infer_256_f16", "infer", "prepared", 8, 128, 256, 256, 5, 3, "f16"),
        # the headline training step: stage 1, float32, three levels
        _case("train_stage1_f32", "train", "prepared", 64, 96, 56, 56, 5, 3, "f32"),
        # mixed-precision training of stage 1 with the deepest pyramid the plane has
        _case("train_stage1_bf16_deep", "train", "prepared", 128, 96, 56, 56, 5, 5, "bf16"),
        # stage 2 through the module, as a network's training loop runs it
        _case("train_stage2_f32", "train", "module", 64, 192, 28, 28, 5, 3, "f32", True),
        # stage 3: many small planes whose rows are not a multiple of four
        _case("train_stage3_bf16", "train", "module", 128, 384, 14, 14, 5, 2, "bf16", True),
        # stage 4: the smallest planes and the most channels
        _case("train_stage4_f32", "train", "prepared", 128, 768, 7, 7, 5, 1, "f32"),
        # odd, non-square planes (detection and segmentation crops)
        _case("train_odd_63x95_f32", "train", "module", 32, 128, 63, 95, 5, 3, "f32", True),
        # planes beyond one compute unit's memory, the largest case
        _case("train_224_f32", "train", "prepared", 16, 64, 224, 224, 5, 3, "f32"),
        # the paper's smaller kernel on its smallest sweep plane, half precision
        _case("train_k3_128_f16", "train", "prepared", 8, 64, 128, 128, 3, 2, "f16"),
        # the paper's larger kernel on a stage-1 plane
        _case("train_k7_56_f32", "train", "prepared", 32, 96, 56, 56, 7, 2, "f32"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    task = "train" if rng.random() < 0.65 else "infer"
    api = rng.choice(["prepared", "module"] if task == "train" else ["prepared", "call"])
    k = rng.choice([5, 5, 5, 3, 7])
    L = rng.randint(1, 5)
    H = _log_uniform(rng, 7, 256)
    W = H if rng.random() < 0.5 else min(256, max(7, int(round(H * rng.uniform(0.6, 1.6)))))
    C = _log_uniform(rng, 16, 512)
    # the largest tensors stay below the largest listed case's, the smallest are a single image
    cap = 30e6 * 25 / max(k * k, 25)
    B = _log_uniform(rng, 1, 128)
    B = max(1, min(B, int(cap / (C * H * W))))
    return {"task": task, "api": api, "B": B, "C": C, "H": H, "W": W, "k": k, "L": L,
            "dtype": rng.choice(["f32", "f32", "bf16", "bf16", "f16"]),
            "bias": api != "prepared" and rng.random() < 0.5}


def _inputs(case, seed):
    """Seeded inputs with the distributions of the package's input recipe: x and dy ~ N(0, 1) in the storage
    type; kernels ~ U(-0.2, 0.2), base scale ~ U(0.5, 1.5), level scales ~ U(0.05, 0.2), bias ~ U(-0.5, 0.5)."""
    g = torch.Generator(device=DEVICE)
    g.manual_seed(1000003 * seed + 17)
    B, C, H, W, k, L = (case[n] for n in "BCHWkL")
    dt = DTYPES[case["dtype"]]

    def normal():
        return torch.randn((B, C, H, W), generator=g, device=DEVICE).to(dt)

    def uniform(shape, lo, hi):
        return torch.rand(shape, generator=g, device=DEVICE) * (hi - lo) + lo

    s = {"x": normal(), "base_w": uniform((C, k, k), -0.2, 0.2), "base_scale": uniform((C,), 0.5, 1.5),
         "level_w": [uniform((4 * C, k, k), -0.2, 0.2) for _ in range(L)],
         "level_scale": [uniform((4 * C,), 0.05, 0.2) for _ in range(L)],
         "bias": uniform((C,), -0.5, 0.5) if case["bias"] else None}
    s["dy"] = normal() if case["task"] == "train" else None
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    params = (s["base_w"], s["base_scale"], s["level_w"], s["level_scale"])
    if case["api"] == "prepared":
        s["fwd"] = binding.Forward(s["x"], *params)
        s["y"] = torch.empty_like(s["x"])
        if case["task"] == "train":
            s["bwd"] = binding.Backward(s["x"], *params)
    elif case["api"] == "module":
        layer = autograd.WTConv2d(case["C"], case["k"], case["L"], bias=case["bias"], device=DEVICE)
        with torch.no_grad():
            layer.base_w.copy_(s["base_w"])
            layer.base_scale.copy_(s["base_scale"])
            if case["bias"]:
                layer.base_bias.copy_(s["bias"])
            for dst, src in zip(list(layer.level_w) + list(layer.level_scale), s["level_w"] + s["level_scale"]):
                dst.copy_(src)
        s["layer"] = layer
        s["x"].requires_grad_(True)
    return s


def run(s):
    case = s["case"]
    if case["api"] == "call":
        return {"y": binding.forward(s["x"], s["base_w"], s["base_scale"], s["level_w"], s["level_scale"],
                                     bias=s["bias"])}
    if case["api"] == "prepared":
        out = {"y": s["fwd"].run(s["x"], s["y"])}
        if case["task"] == "train":
            b = s["bwd"]
            b.run(s["x"], s["dy"])
            out.update(dx=b.dx, d_base_w=b.dbw, d_base_scale=b.dbs, d_level_w=b.dlw, d_level_scale=b.dls)
        return out
    layer, x = s["layer"], s["x"]
    x.grad = None
    layer.zero_grad(set_to_none=True)
    y = layer(x)
    y.backward(s["dy"])
    out = {"y": y.detach(), "dx": x.grad, "d_base_w": layer.base_w.grad, "d_base_scale": layer.base_scale.grad,
           "d_level_w": [p.grad for p in layer.level_w], "d_level_scale": [p.grad for p in layer.level_scale]}
    if layer.base_bias is not None:
        out["d_bias"] = layer.base_bias.grad
    return out


def work(case):
    """Bytes: x read, y written, and for a training step x and dy read and dx written, with the parameters and
    their gradients. Operations: two per multiply-add of the base kernel and of every subband kernel, once for
    the forward and twice more for the backward (dx and the kernel gradients)."""
    B, C, H, W, k, L = (case[n] for n in "BCHWkL")
    n = B * C * H * W
    sites = n
    h, w = H, W
    for _ in range(L):
        h, w = (h + 1) // 2, (w + 1) // 2
        sites += 4 * B * C * h * w
    params = 4 * C * (1 + 4 * L) * (k * k + 1)
    e = 4 if case["dtype"] == "f32" else 2
    train = case["task"] == "train"
    return {"bytes": (5 if train else 2) * n * e + (2 if train else 1) * params,
            "flops": 2 * k * k * sites * (3 if train else 1)}


def tolerance(case):
    # Largest relative error over all outputs; 16-bit outputs are dominated by their own rounding, and by that
    # of the coarse carriers of large planes, which are held in the storage type.
    return {"rel": {"f32": 2e-6, "bf16": 1e-2, "f16": 1.5e-3}[case["dtype"]]}


# ---------------------------------------------------------------------------
# the operator in 64 bits, step by step (Haar analysis with zero padding,
# depthwise correlation per subband, scale, synthesis with cropping)
# ---------------------------------------------------------------------------
def _conv(x, w):
    k = w.shape[-1]
    H, W = x.shape[-2:]
    xp = F.pad(x, [k // 2] * 4)
    out = torch.zeros_like(x)
    for p in range(k):
        for t in range(k):
            out.addcmul_(xp[..., p:p + H, t:t + W], w[:, p, t].view(1, -1, 1, 1))
    return out


def _conv_grad(dz, x, k):
    """Gradient of _conv's kernel for the upstream gradient dz."""
    H, W = x.shape[-2:]
    xp = F.pad(x, [k // 2] * 4)
    return torch.stack([torch.stack([(dz * xp[..., p:p + H, t:t + W]).sum((0, 2, 3)) for t in range(k)], -1)
                        for p in range(k)], -2)


def _analysis(x):
    """One orthonormal Haar level of the zero-padded planes: [B, C, H, W] -> [B, 4C, h, w], channel 4c + band."""
    B, C, H, W = x.shape
    x = F.pad(x, [0, W % 2, 0, H % 2])
    a, b = x[..., 0::2, 0::2], x[..., 0::2, 1::2]
    c, d = x[..., 1::2, 0::2], x[..., 1::2, 1::2]
    y = torch.stack([a + b + c + d, a + b - c - d, a - b + c - d, a - b - c + d], 2) / 2
    return y.reshape(B, 4 * C, *y.shape[-2:])


def _synthesis(z, H, W):
    """Inverse (and adjoint) of _analysis, cropped to H x W."""
    B, C4, h, w = z.shape
    ll, lh, hl, hh = z.view(B, C4 // 4, 4, h, w).unbind(2)
    out = z.new_empty(B, C4 // 4, 2 * h, 2 * w)
    out[..., 0::2, 0::2] = (ll + lh + hl + hh) / 2
    out[..., 0::2, 1::2] = (ll + lh - hl - hh) / 2
    out[..., 1::2, 0::2] = (ll - lh + hl - hh) / 2
    out[..., 1::2, 1::2] = (ll - lh - hl + hh) / 2
    return out[..., :H, :W]


def _branch(x, ws):
    """Haar branch of Algorithm 1 for folded kernels ws; also every level's coefficients."""
    ys, sizes, cur = [], [], x
    for _ in ws:
        sizes.append(cur.shape[-2:])
        ys.append(_analysis(cur))
        cur = ys[-1][:, 0::4]
    r = None
    for y, w, (H, W) in reversed(list(zip(ys, ws, sizes))):
        z = _conv(y, w)
        if r is not None:
            z[:, 0::4] += r
        r = _synthesis(z, H, W)
    return r, ys


def exact(case, seed):
    s = _inputs(case, seed)
    k = case["k"]
    x = s["x"].double()
    w0, s0 = s["base_w"].double(), s["base_scale"].double()
    lw, ls = [w.double() for w in s["level_w"]], [v.double() for v in s["level_scale"]]
    b0 = s["bias"].double() if s["bias"] is not None else torch.zeros_like(s0)
    folded = [w * v.view(-1, 1, 1) for w, v in zip(lw, ls)]
    r, ys = _branch(x, folded)
    y = _conv(x, w0 * s0.view(-1, 1, 1)) + (s0 * b0).view(1, -1, 1, 1) + r
    out = {"y": y}
    if case["task"] != "train":
        return out
    dy = s["dy"].double()
    # the adjoint of a correlation is the correlation with the rotated kernel, and synthesis and analysis are
    # each other's transposes
    rd, dys = _branch(dy, [w.flip(-1, -2) for w in folded])
    out["dx"] = _conv(dy, (w0 * s0.view(-1, 1, 1)).flip(-1, -2)) + rd
    g0 = _conv_grad(dy, x, k)
    sdy = dy.sum((0, 2, 3))
    out["d_base_w"] = g0 * s0.view(-1, 1, 1)
    out["d_base_scale"] = (g0 * w0).sum((1, 2)) + b0 * sdy
    gl = [_conv_grad(dz, yl, k) for dz, yl in zip(dys, ys)]
    out["d_level_w"] = [g * v.view(-1, 1, 1) for g, v in zip(gl, ls)]
    out["d_level_scale"] = [(g * w).sum((1, 2)) for g, w in zip(gl, lw)]
    if case["bias"]:
        out["d_bias"] = s0 * sdy
    return out
