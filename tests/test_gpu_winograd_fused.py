"""The one-kernel Winograd convolution: each block shape where it can go wrong
(ragged blocks of tiles and channels, a stage of 16 channels that ends early,
one stage and several, output channels that break 16-byte stores, asymmetric and
no padding, tiles that span images), against the three-kernel form's oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_1904_05347_amd import workloads as wl
from .gpu_util import assert_parity, dev, host, require_gpu
from .test_gpu_winograd import _check_integers, _scale

pytestmark = pytest.mark.gpu

# tile, (N, H, W, Cin, Cout, pads), the form the prediction picks
CASES = [
    (2, (2, 9, 11, 20, 24, (1, 1, 1, 1)), "winograd2_32x32"),
    (2, (5, 13, 7, 4, 33, (0, 2, 1, 0)), "winograd2_32x32"),
    (2, (3, 16, 18, 52, 65, (0, 0, 0, 0)), "winograd2_32x32"),
    (2, (1, 249, 250, 12, 61, (1, 1, 1, 1)), "winograd2_32x64"),
    (4, (3, 43, 39, 12, 43, (1, 1, 1, 1)), "winograd4_32x32"),
    (4, (2, 230, 227, 16, 61, (2, 1, 0, 1)), "winograd4_32x64"),
]


@pytest.mark.parametrize("tile,geom,form", CASES, ids=["F%d_%s" % (t, "x".join(map(str, g[:5]))) for t, g, _ in CASES])
def test_winograd_one_kernel_forms(tile, geom, form):
    torch, pk = require_gpu()
    N, H, W, Cin, Cout, pads = geom
    rng = np.random.default_rng(sum(geom[:5]) + tile)
    Ho, Wo = oracle.conv2d_out_dims(H, W, 3, 3, 1, 1, *pads)
    for kind in ("uniform", "int"):
        draw = wl.uniform if kind == "uniform" else wl.integers
        x = draw(rng, N * H * W * Cin).reshape(N, H, W, Cin)
        f = draw(rng, 9 * Cin * Cout).reshape(3, 3, Cin, Cout)
        # NaN behind the image: nothing past it is read into a result
        flat = torch.full((x.size + 64,), float("nan"), dtype=torch.float32, device="cuda")
        dx = flat[:x.size].view(x.shape)
        dx.copy_(dev(x))
        outs = []
        for _ in range(2):
            y = torch.full((N, Ho, Wo, Cout), float("nan"), dtype=torch.float32, device="cuda")
            ws = torch.full((pk.conv2d_winograd_workspace_bytes(N, H, W, Cin, Cout, *pads, tile) // 4,), float("nan"),
                            dtype=torch.float32, device="cuda")
            pk.conv2d_winograd(dx, dev(f), padding=pads, out=y, workspace=ws, tile=tile)
            assert pk.last_config_name() == form
            outs.append(host(y))
        assert np.array_equal(outs[0], outs[1])
        ref, _ = oracle.conv2d(x, f, (1, 1), pads)
        what = "F(%d) %s" % (tile, geom)
        if kind == "int":
            _check_integers(tile, outs[0], ref, _scale(tile, x, f, pads), what)
        else:
            assert_parity(outs[0], ref, _scale(tile, x, f, pads), what)
