"""The predicted choice of tile and split for shapes outside the table (host
only): every tile it names is compiled, and no split asks for more partial sums
than the static scratch of the no-allocation entry holds."""
import os
import random
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def pk():
    import paper_1904_05347_amd as pk
    pk.load()
    return pk


def test_cost_tiles_are_compiled(pk):
    names = {c["name"]: c for c in pk.configs()}
    src = open(os.path.join(ROOT, "paper_1904_05347_amd", "csrc", "pk_cost.hpp")).read()
    rows = re.findall(r'\{"((?:gemm|conv)_[a-z0-9_%]+)", (\d+), (\d+), (\d+), (\d+), (\d+), (\d)', src)
    assert len(rows) >= 40
    for name, bm, bn, bk, kg, per_cu, sk in rows:
        for lay in ("nn", "nt", "tn", "tt") if "%s" in name else ("",):
            n = name % lay if lay else name
            if n not in names:  # aligned TN keeps its register-staged 32-row form
                assert n == "gemm_32x64x32_w1x2_k4_tn_v44_dma3", n
                continue
            c = names[n]
            assert (c["bm"], c["bn"], c["bk"], c["kgroups"], c["streamk"]) == tuple(map(int, (bm, bn, bk, kg, sk))), n
            assert int(per_cu) * c["lds_bytes"] <= 160 * 1024 and int(per_cu) * c["threads"] <= 2048, n


def test_chosen_partial_sums_fit_the_static_scratch(pk):
    rng = random.Random(7)
    for _ in range(3000):
        n, h, w = rng.randint(1, 64), rng.randint(7, 256), rng.randint(7, 256)
        cin, cout, k, s = rng.randint(1, 2048), rng.randint(1, 2048), rng.choice([1, 3, 5, 7]), rng.choice([1, 2])
        need = pk.conv2d_workspace_bytes(n, h, w, cin, k, k, cout, s, s, *pk.conv2d_same_pads(h, w, k, k, s, s))
        assert need <= pk.binding.NOALLOC_SCRATCH_BYTES, (n, h, w, cin, cout, k, s, need)
