"""The configuration and split of a call do not depend on whether its workspace
is just what the size query asked or larger: the sizes here are ones where the
older rule's split needs more room than the chosen one's, and where judging by
the room alone took another tile or split."""
from __future__ import annotations

import pytest

from .gpu_util import require_gpu

pytestmark = pytest.mark.gpu

# M, N, K, trans_a, trans_b
GEMMS = [(1493, 421, 6904, True, True), (431, 1293, 7423, False, False)]
# N, H, W, Cin, window, Cout
CONVS = [(1, 88, 88, 308, 3, 219), (1, 180, 180, 379, 3, 16), (1, 150, 150, 188, 3, 112), (1, 128, 128, 428, 3, 40)]


def _same(torch, pk, call):
    y = call(None)
    name = pk.last_config_name()
    z = call(torch.empty(32 << 20, dtype=torch.float32, device="cuda"))
    assert pk.last_config_name() == name
    assert torch.equal(y, z)  # the same additions in the same order


@pytest.mark.parametrize("M,N,K,ta,tb", GEMMS)
def test_gemm_choice_at_queried_workspace(M, N, K, ta, tb):
    torch, pk = require_gpu()
    a = torch.randn((K, M) if ta else (M, K), device="cuda")
    b = torch.randn((N, K) if tb else (K, N), device="cuda")
    _same(torch, pk, lambda ws: pk.gemm(a, b, trans_a=ta, trans_b=tb, workspace=ws))


@pytest.mark.parametrize("n,h,w,cin,k,cout", CONVS)
def test_conv_choice_at_queried_workspace(n, h, w, cin, k, cout):
    torch, pk = require_gpu()
    x = torch.randn((n, h, w, cin), device="cuda")
    f = torch.randn((k, k, cin, cout), device="cuda")
    _same(torch, pk, lambda ws: pk.conv2d_fwd(x, f, workspace=ws))


@pytest.mark.parametrize("M,N,K", [(12, 6920, 796), (284, 1996, 2776)])
def test_sliced_gemm_choice_at_its_own_workspace(M, N, K):
    """Operands inside wider rows get the workspace of their own choice."""
    torch, pk = require_gpu()
    a = torch.randn((K, M + 3), device="cuda")[:, :M]
    b = torch.randn((N, K + 3), device="cuda")[:, :K]
    _same(torch, pk, lambda ws: pk.gemm(a, b, trans_a=True, trans_b=True, workspace=ws))


@pytest.mark.parametrize("n,h,w,cin,cout", [(1, 56, 57, 460, 288), (2, 30, 31, 324, 52)])
def test_conv_choice_at_4_byte_addresses(n, h, w, cin, cout):
    """... and an image and a filter at addresses aligned to 4 bytes only."""
    torch, pk = require_gpu()
    x = torch.randn(1 + n * h * w * cin, device="cuda")[1:].view(n, h, w, cin)
    f = torch.randn(1 + 9 * cin * cout, device="cuda")[1:].view(3, 3, cin, cout)
    _same(torch, pk, lambda ws: pk.conv2d_fwd(x, f, workspace=ws))
