"""The calls whose time is followed from change to change.

Each case is one call of the package's public entry points (``gemm``,
``conv2d_fwd``, ``conv2d_winograd``) as a program makes it: operands resident
on the GPU, output and workspace left to the call.  ``listed`` names twelve of
them, ``draw`` makes further ones of the same ranges:

- matrix products of all four layouts, from 16 to 4096 on a side, aligned and
  odd sizes, operands that are slices of wider arrays, with and without the
  accumulation beta * C, and the few-row products of a dense layer at small
  batch;
- convolutions with 1x1 to 7x7 windows, stride 1 and 2, batch 1 to 32, three
  input channels to 1024, channel counts that are no multiple of four, square
  and other images, same and no padding;
- Winograd convolutions with both output-tile sizes.
"""
import math

import torch

import paper_1904_05347_amd as pk


# ------------------------------------------------------------------ the cases

def _gemm(name, M, N, K, ta=False, tb=False, beta=0.0, slack=0):
    return {"name": name, "op": "gemm", "M": M, "N": N, "K": K, "ta": ta, "tb": tb, "beta": beta, "slack": slack}


def _conv(name, n, h, w, cin, k, cout, stride=1, same=True):
    return {"name": name, "op": "conv", "n": n, "h": h, "w": w, "cin": cin, "k": k, "cout": cout,
            "stride": stride, "same": same}


def _wino(name, n, h, w, cin, cout, tile):
    return {"name": name, "op": "winograd", "n": n, "h": h, "w": w, "cin": cin, "cout": cout, "tile": tile}


def listed():
    return [
        # the smallest product of the power-of-two sweep: launch latency and host work
        _gemm("gemm_64", 64, 64, 64),
        # the middle of that sweep: few tiles, a short reduction
        _gemm("gemm_512x1024x256", 512, 1024, 256),
        # a dense layer at batch 32 on weights stored output-major: the weights are read once
        _gemm("gemm_dense_b32", 32, 4096, 4096, tb=True),
        # a weight gradient of odd sizes added to what is there, both operands slices of wider arrays
        _gemm("gemm_odd_tn_acc", 1021, 1531, 1777, ta=True, beta=0.5, slack=3),
        # the large square product
        _gemm("gemm_4096", 4096, 4096, 4096),
        # a deep layer of the VGG-16 table for one image: few outputs, a long reduction
        _conv("conv_14x14x512_b1", 1, 14, 14, 512, 3, 512),
        # a 1x1 layer of the ResNet-50 table at small batch
        _conv("conv_1x1_28x28x512_b4", 4, 28, 28, 512, 1, 128),
        # ResNet-50's first layer: three channels, 7x7, stride 2, no padding
        _conv("conv_stem_b32", 32, 230, 230, 3, 7, 64, stride=2, same=False),
        # channel counts that no vector width divides, an image that is not square
        _conv("conv_odd_channels_b8", 8, 57, 43, 50, 3, 75),
        # a large 3x3 layer of the VGG-16 table at batch 32
        _conv("conv_28x28x256_b32", 32, 28, 28, 256, 3, 512),
        # Winograd with the small tile where a net begins, few images
        _wino("wino2_56x56x64_b4", 4, 56, 56, 64, 64, 2),
        # Winograd with the large tile at batch 32, where it is worth most
        _wino("wino4_56x56x256_b32", 32, 56, 56, 256, 256, 4),
    ]


MOST_FLOPS = 6.0e10   # of a drawn case: below the largest listed ones
MOST_BYTES = 4.5e8


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """Half of the sizes as they fall, odd ones among them, half rounded to a multiple of 32, 16 or 4."""
    v = _log(rng, lo, hi)
    if rng.random() < 0.5:
        step = rng.choice([s for s in (32, 16, 4) if s <= max(v, 4)] or [4])
        v = max(step, int(round(v / step)) * step)
    return min(max(v, lo), hi)


def _draw_one(rng):
    kind = rng.choice(["gemm", "gemm", "gemm", "dense", "conv", "conv", "conv", "winograd", "winograd"])
    if kind == "gemm":
        return {"op": "gemm", "M": _size(rng, 16, 4096), "N": _size(rng, 16, 4096), "K": _size(rng, 16, 4096),
                "ta": rng.random() < 0.5, "tb": rng.random() < 0.5, "beta": rng.choice([0.0, 0.0, 0.5, 1.0]),
                "slack": rng.choice([0, 0, 0, 4, 3])}
    if kind == "dense":
        return {"op": "gemm", "M": _log(rng, 1, 64), "N": _size(rng, 512, 8192), "K": _size(rng, 512, 8192),
                "ta": False, "tb": rng.random() < 0.7, "beta": 0.0, "slack": 0}
    h = _log(rng, 7, 224)
    w = h if rng.random() < 0.6 else max(7, min(224, int(h * rng.uniform(0.6, 1.6))))
    cin = 3 if kind == "conv" and rng.random() < 0.2 else _size(rng, 8, 1024)
    if kind == "conv":
        return {"op": "conv", "n": _log(rng, 1, 32), "h": h, "w": w, "cin": cin, "k": rng.choice([1, 1, 3, 3, 5, 7]),
                "cout": _size(rng, 8, 1024), "stride": rng.choice([1, 1, 2]), "same": rng.random() < 0.8}
    return {"op": "winograd", "n": _log(rng, 1, 32), "h": h, "w": w, "cin": cin, "cout": _size(rng, 8, 1024),
            "tile": rng.choice([2, 4])}


def draw(rng):
    while True:
        c = _draw_one(rng)
        w = work(c)
        if w["flops"] <= MOST_FLOPS and w["bytes"] <= MOST_BYTES:
            return c


# ------------------------------------------------------------------ geometry

def _geometry(c):
    """(window, stride, pads top/left/bottom/right, Ho, Wo) of a convolution."""
    k, s = c.get("k", 3), c.get("stride", 1)
    h, w = c["h"], c["w"]
    if not c.get("same", True):
        return k, s, (0, 0, 0, 0), (h - k) // s + 1, (w - k) // s + 1
    ho, wo = -(-h // s), -(-w // s)
    ph, pw = max(0, (ho - 1) * s + k - h), max(0, (wo - 1) * s + k - w)
    return k, s, (ph // 2, pw // 2, ph - ph // 2, pw - pw // 2), ho, wo


def work(case):
    if case["op"] == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": 4 * (M * K + K * N + M * N * (2 if case["beta"] else 1)), "flops": 2 * M * N * K}
    k, s, _, ho, wo = _geometry(case)
    n, h, w, cin, cout = case["n"], case["h"], case["w"], case["cin"], case["cout"]
    read = n * cin * (ho * wo if k == 1 else h * w)  # a strided 1x1 window skips pixels
    flops = 2 * n * ho * wo * cout * k * k * cin
    if case["op"] == "winograd":
        # the multiplications of the batched products: (m + 2)^2 for m * m outputs and nine taps
        m = case["tile"]
        flops = 2 * n * -(-ho // m) * -(-wo // m) * (m + 2) ** 2 * cin * cout
    return {"bytes": 4 * (read + k * k * cin * cout + n * ho * wo * cout), "flops": flops}


# ------------------------------------------------------------------ inputs

def _matrix(g, rows, cols, slack, scale=1.0):
    t = torch.randn((rows, cols + slack), generator=g, device="cuda") * scale
    return t[:, :cols]


def prepare(case, seed):
    """Activations (rectified before a convolution) and weights scaled to keep their variance."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    if case["op"] == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        a = _matrix(g, *((K, M) if case["ta"] else (M, K)), case["slack"])
        b = _matrix(g, *((N, K) if case["tb"] else (K, N)), case["slack"], K ** -0.5)
        c = torch.randn((M, N), generator=g, device="cuda") if case["beta"] else None
        return {"case": case, "a": a, "b": b, "c": c}
    k = case.get("k", 3)
    x = torch.randn((case["n"], case["h"], case["w"], case["cin"]), generator=g, device="cuda").relu_()
    w = torch.randn((k, k, case["cin"], case["cout"]), generator=g, device="cuda")
    return {"case": case, "x": x, "w": w * (2.0 / (k * k * case["cin"])) ** 0.5}


def run(state):
    case = state["case"]
    if case["op"] == "gemm":
        # the product is added to a copy: the state's own C serves every pass
        c = state["c"].clone() if case["beta"] else None
        return pk.gemm(state["a"], state["b"], c, beta=case["beta"], trans_a=case["ta"], trans_b=case["tb"])
    if case["op"] == "winograd":
        return pk.conv2d_winograd(state["x"], state["w"], padding="SAME", tile=case["tile"])
    return pk.conv2d_fwd(state["x"], state["w"], stride=case["stride"], padding="SAME" if case["same"] else "VALID")


# ------------------------------------------------------------------ results

def tolerance(case):
    """About four times the distance of the 32-bit sums from the 64-bit ones, which was
    1.1e-6 on the longest reductions, 2.6e-6 with the large Winograd tile and up to 7e-7 otherwise."""
    if case["op"] == "winograd":
        return {"rel": 1e-5 if case["tile"] == 4 else 3e-6}
    return {"rel": 5e-6}


def exact(case, seed):
    s = prepare(case, seed)
    if case["op"] == "gemm":
        a, b = s["a"].double(), s["b"].double()
        r = (a.t().contiguous() if case["ta"] else a.contiguous()) @ (b.t().contiguous() if case["tb"] else b.contiguous())
        return r + case["beta"] * s["c"].double() if case["beta"] else r
    k, st, (pt, pl, pb, pr), ho, wo = _geometry(case)
    x, w = s["x"].double(), s["w"].double()
    x = torch.nn.functional.pad(x, (0, 0, pl, pr, pt, pb))
    y = torch.zeros((case["n"] * ho * wo, case["cout"]), dtype=torch.float64, device=x.device)
    for i in range(k):
        for j in range(k):
            tap = x[:, i:i + (ho - 1) * st + 1:st, j:j + (wo - 1) * st + 1:st, :].reshape(-1, case["cin"])
            y.addmm_(tap, w[i, j])
    return y.reshape(case["n"], ho, wo, case["cout"])
