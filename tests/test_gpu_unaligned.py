"""The direct-to-LDS forms for operands of any 4-byte alignment, size and
leading dimension: integer data, so every output must equal the oracle bit for
bit; the columns between a row's end and its leading dimension, and the
elements around the operand, hold NaN, so an element read past a row, past K or
past the operand shows."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_1904_05347_amd import workloads as wl
from .gpu_util import dev, host, require_gpu

pytestmark = pytest.mark.gpu


def _inside_nan(torch, a, slack):
    """a as a view of a NaN-filled allocation: one element before it, slack
    columns after every row but the last, nothing after the last element."""
    r, c = a.shape
    flat = torch.full((1 + (r - 1) * (c + slack) + c,), float("nan"), dtype=torch.float32, device="cuda")
    v = flat[1:].as_strided((r, c), (c + slack, 1))
    v.copy_(dev(a))
    return v


def _unaligned(pk, kind):
    return [c["name"] for c in pk.configs() if c["kind"] == kind and c["dma"] and ("_v11" in c["name"] or "_v41" in c["name"])]


# one element; a tile edge each way; K one short of, at and past a K-block; K a
# multiple of four behind an odd leading dimension; several ragged tiles
GEMM_SHAPES = [(1, 1, 1, 0), (33, 129, 31, 3), (129, 33, 32, 1), (65, 97, 33, 2), (97, 65, 68, 1), (257, 130, 333, 3)]


@pytest.mark.parametrize("M,N,K,slack", GEMM_SHAPES, ids=["%dx%dx%d+%d" % s for s in GEMM_SHAPES])
def test_gemm_unaligned_configs(M, N, K, slack):
    torch, pk = require_gpu()
    infos = {c["name"]: c for c in pk.configs()}
    ran = 0
    for name in _unaligned(pk, 0):
        ta, tb = infos[name]["trans_a"], infos[name]["trans_b"]
        rng = np.random.default_rng(M * 5 + N * 3 + K)
        A = wl.integers(rng, M * K).reshape((K, M) if ta else (M, K))
        B = wl.integers(rng, K * N).reshape((N, K) if tb else (K, N))
        C = wl.integers(rng, M * N).reshape(M, N)
        ref, _ = oracle.sgemm("NT"[ta], "NT"[tb], M, N, K, 1.0, A, A.shape[1], B, B.shape[1], 0.5, C, N)
        dA, dB = _inside_nan(torch, A, slack), _inside_nan(torch, B, slack)
        ws = torch.empty(2 * M * N, dtype=torch.float32, device="cuda")
        for splits in (1, 2):
            dC = _inside_nan(torch, C, slack)
            pk.force_config(name)
            pk.force_splits(splits)
            try:
                pk.gemm(dA, dB, dC, beta=0.5, trans_a=bool(ta), trans_b=bool(tb), workspace=ws)
                assert pk.last_config_name() == name
            finally:
                pk.force_config(None)
                pk.force_splits(0)
            assert np.array_equal(host(dC).astype(np.float64), ref), (name, splits)
            ran += 1
    assert ran >= 2 * 4 * 10


# N, H, W, Cin, KH, KW, Cout, stride, pads: fewer channels than a chunk, a
# K-block that ends inside a tap, several taps per K-block, windows that are
# not square, strides with asymmetric padding, a strided 1x1
CONV_GEOMS = [
    (2, 9, 11, 3, 3, 3, 7, (1, 1), (1, 1, 1, 1)), (1, 13, 7, 1, 5, 2, 33, (2, 1), (2, 0, 1, 1)),
    (3, 8, 9, 50, 3, 3, 75, (1, 1), (1, 1, 1, 1)), (2, 15, 15, 37, 1, 1, 130, (2, 2), (0, 0, 0, 0)),
    (2, 10, 12, 20, 3, 3, 97, (2, 2), (0, 0, 1, 1)), (1, 6, 6, 129, 7, 7, 5, (1, 1), (3, 3, 3, 3)),
]


@pytest.mark.parametrize("geom", CONV_GEOMS, ids=lambda g: "x".join(map(str, g[:7])))
def test_conv_unaligned_configs(geom):
    torch, pk = require_gpu()
    N, H, W, Cin, KH, KW, Cout, stride, pads = geom
    rng = np.random.default_rng(sum(geom[:7]))
    x = wl.integers(rng, N * H * W * Cin).reshape(N, H, W, Cin)
    f = wl.integers(rng, KH * KW * Cin * Cout).reshape(KH, KW, Cin, Cout)
    ref, _ = oracle.conv2d(x, f, stride, pads)
    dx = _inside_nan(torch, x.reshape(1, -1), 0).view(x.shape)
    df = _inside_nan(torch, f.reshape(1, -1), 0).view(f.shape)
    dx4 = dev(x)  # 16-byte aligned, for the forms that ask it of the image
    ws = torch.empty(2 * ref.size, dtype=torch.float32, device="cuda")
    ran = 0
    for name in _unaligned(pk, 1):
        if "_v41" in name and Cin % 4:
            continue
        for splits in (1, 2):
            y = torch.full(ref.shape, float("nan"), dtype=torch.float32, device="cuda")
            pk.force_config(name)
            pk.force_splits(splits)
            try:
                pk.conv2d_fwd(dx4 if "_v41" in name else dx, df, stride=stride, padding=pads, out=y, workspace=ws)
                assert pk.last_config_name() == name
            finally:
                pk.force_config(None)
                pk.force_splits(0)
            assert np.array_equal(host(y).astype(np.float64), ref), (name, splits)
            ran += 1
    assert ran >= 14


# one element, a ragged last work-group, one column, rows aligned but not C's;
# the largest result summed one element per work-item, and beyond it four
# elements each: a last work-item of four, three, two and one, rows of one, two,
# three and five
@pytest.mark.parametrize("M,N", [(1, 1), (3, 1), (1, 3), (192, 23), (37, 31), (16, 24), (1 << 14, 16), (87382, 3),
                                 (1031, 255), (262147, 1), (131073, 2), (262145, 1),
                                 (65537, 4), (52430, 5), (517, 509)])
@pytest.mark.parametrize("splits", [2, 9, 16])
def test_splitk_sum_of_rows_of_any_length(M, N, splits):
    torch, pk = require_gpu()
    K = 16 * 32 if M * N < 1000 else 16 * 16
    rng = np.random.default_rng(M * 7 + N + splits)
    A, B, C = (wl.integers(rng, r * c).reshape(r, c) for r, c in ((M, K), (K, N), (M, N)))
    ws = torch.full((splits * M * N,), float("nan"), dtype=torch.float32, device="cuda")
    pk.force_config("gemm_64x64x16_w2x2_nn_v11_dma3")
    pk.force_splits(splits)
    try:
        ref0, _ = oracle.sgemm("N", "N", M, N, K, 1.0, A, K, B, N, 0.0, None, N)
        for beta, slack in ((0.0, 0), (0.5, 0), (0.0, 3), (0.5, 2)):
            dC = _inside_nan(torch, C, slack)
            if beta == 0.0:
                dC.fill_(float("nan"))
            pk.gemm(dev(A), dev(B), dC, beta=beta, workspace=ws)
            ref = ref0 + beta * C.astype(np.float64)  # exact on these integers
            assert np.array_equal(host(dC).astype(np.float64), ref), (beta, slack)
            if slack and M > 1:  # what lies between the rows stays
                gap = dC.as_strided((M - 1, slack), (N + slack, 1), dC.storage_offset() + N)
                assert bool(torch.isnan(gap).all())
    finally:
        pk.force_config(None)
        pk.force_splits(0)


def test_conv_unaligned_infinities_stay_in_their_windows():
    """An infinity or NaN in the image reaches exactly the outputs whose window
    holds it."""
    torch, pk = require_gpu()
    rng = np.random.default_rng(3)
    N, H, W, Cin, Cout = 2, 9, 10, 5, 7
    f = np.abs(wl.uniform(rng, 9 * Cin * Cout)).reshape(3, 3, Cin, Cout) + np.float32(0.5)
    for value in (np.inf, np.nan):
        for n, h, w, c in [(0, 4, 5, 0), (1, 8, 9, 4), (1, 0, 0, 2), (0, 3, 9, 1)]:
            x = np.zeros((N, H, W, Cin), np.float32)
            x[n, h, w, c] = value
            hit = np.zeros((N, H, W), bool)
            hit[n, max(0, h - 1):h + 2, max(0, w - 1):w + 2] = True
            for name in [q for q in _unaligned(pk, 1) if "_v11" in q]:
                pk.force_config(name)
                try:
                    y = host(pk.conv2d_fwd(dev(x), dev(f)))
                finally:
                    pk.force_config(None)
                assert np.array_equal(~np.isfinite(y).all(axis=-1), hit), (name, value, n, h, w, c)
                assert np.all(y[~hit] == 0), (name, value)


def test_narrow_tile_swizzle_and_tt():
    """The 32- and 96-column tiles (k rows swapped in pairs) and the TT forms
    on aligned operands, several K-blocks deep, every column distinct."""
    torch, pk = require_gpu()
    ran = 0
    for c in pk.configs():
        if c["kind"] != 0 or not c["dma"] or "_v44" not in c["name"] or c["streamk"]:
            continue
        if not (c["trans_a"] and c["trans_b"]) and c["bn"] not in (32, 96) and c["bm"] != 32:
            continue
        ta, tb = c["trans_a"], c["trans_b"]
        M, N, K = 160, 196, 132
        rng = np.random.default_rng(c["bm"] + c["bn"])
        A = wl.integers(rng, M * K).reshape((K, M) if ta else (M, K))
        B = wl.integers(rng, K * N).reshape((N, K) if tb else (K, N))
        ref, _ = oracle.sgemm("NT"[ta], "NT"[tb], M, N, K, 1.0, A, A.shape[1], B, B.shape[1], 0.0,
                              np.zeros((M, N), np.float32), N)
        dC = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
        pk.force_config(c["name"])
        try:
            pk.gemm(dev(A), dev(B), dC, trans_a=bool(ta), trans_b=bool(tb))
        finally:
            pk.force_config(None)
        assert np.array_equal(host(dC).astype(np.float64), ref), c["name"]
        ran += 1
    assert ran >= 20
