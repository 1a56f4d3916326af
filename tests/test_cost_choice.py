"""The predicted choice of tile and split for shapes outside the table (host
only): every tile it names is compiled, no split asks for more partial sums
than the static scratch of the no-allocation entry holds, and no choice has a
longer chain of additions than the rule's."""
import ctypes
import math
import os
import random
import re
import subprocess

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


class _Pick(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int64) for n in ("bm", "bn", "bk", "kg", "streamk", "splits")] + [("us", ctypes.c_double)]


@pytest.fixture(scope="module")
def choice(pk, tmp_path_factory):
    """(rule's pick, chosen pick) of a product or a convolution at a workspace size."""
    out = str(tmp_path_factory.mktemp("shim") / "libchoice_shim.so")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "--offload-arch=gfx950", "-x", "hip", "-O1", "-std=c++20", "-shared", "-fPIC",
                    os.path.join(ROOT, "tests", "choice_shim.cpp"), "-o", out, "-L" + os.path.dirname(pk.binding.LIB_PATH),
                    "-l:" + os.path.basename(pk.binding.LIB_PATH),
                    "-Wl,-Bsymbolic", "-Wl,-rpath," + os.path.dirname(pk.binding.LIB_PATH)], check=True, capture_output=True)
    lib = ctypes.CDLL(out)
    i64, sz, p = ctypes.c_int64, ctypes.c_size_t, ctypes.POINTER(_Pick)
    lib.shim_gemm.argtypes = [ctypes.c_int, ctypes.c_int, i64, i64, i64, ctypes.c_int, sz, p, p]
    lib.shim_conv.argtypes = [i64, i64, i64, ctypes.c_int, ctypes.c_int, ctypes.c_int, sz, p, p]

    def call(fn, *args):
        rule, pick = _Pick(), _Pick()
        getattr(lib, fn)(*args, rule, pick)
        return rule, pick

    call.lib = lib
    return call


def test_look_up_by_name_allocates_nothing(pk, choice):
    """The first look-up builds its index without an allocation, whose failure
    would leave the C entry as an exception; every name is found, others not."""
    assert choice.lib.shim_force_without_memory(b"conv_64x64x32_w2x2_v44_dma2") == 0
    assert choice.lib.shim_force_without_memory(b"conv_none") == 1
    for c in pk.configs():
        pk.force_config(c["name"])
    pk.force_config(None)


ALL_ROOM = (1 << 64) - 1


def _chain(c, M, N, K):
    """Longest run of products one accumulator of this pick adds up, in K."""
    nkb = -(-K // c.bk)
    if c.streamk:  # equal shares of all tiles' K-blocks over two work-groups per CU
        blocks = min(nkb, -(-(-(-M // c.bm) * -(-N // c.bn) * nkb) // 512))
    else:
        blocks = -(-(-(-nkb // c.splits)) // c.kg)
    return min(K, blocks * c.bk)


def _chain32(c, M, N, K):
    """... to the end of a K-block of 32."""
    return -(-_chain(c, M, N, K) // 32) * 32


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _products(rng, count):
    """(trans_a, trans_b, M, N, K, 16-byte accesses)"""
    for i in range(count):
        M, N, K = _log(rng, 1, 8192), _log(rng, 16, 8192), _log(rng, 16, 16384)
        if i % 2:
            M, N, K = max(4, M // 4 * 4), N // 4 * 4, K // 4 * 4
        yield rng.randint(0, 1), rng.randint(0, 1), M, N, K, i % 2


# one K-block past a split's whole ones; and of convolutions whose rule is stream-K
PRODUCTS = [(0, 0, 1025, 64, 1025, 0), (0, 0, 64, 64, 1025, 0), (1, 1, 1493, 421, 6904, 0)]
STREAMK_CONVS = [(8, 35, 128, 3, 192, 1), (18, 24, 156, 3, 160, 1), (3, 118, 48, 7, 336, 2), (9, 21, 128, 3, 424, 1)]


def _convs(rng, count):
    """(M, Cout, K, 16-byte image, 16-byte filter, channels multiples of four)"""
    for n, h, cin, k, cout, s in STREAMK_CONVS:
        yield n * (-(-h // s)) ** 2, cout, k * k * cin, 1, 1, 1
    for i in range(count):
        h, s, k = _log(rng, 7, 224), rng.choice([1, 1, 2]), rng.choice([1, 3, 3, 5, 7])
        M, K = _log(rng, 1, 32) * (-(-h // s)) ** 2, k * k * (_log(rng, 8, 1024) // 4 * 4)
        cout = max(4, _log(rng, 8, 1024) // 4 * 4)
        if M * cout * K < 4e10 and M * cout < 1e8:
            yield M, cout, K, i % 4 < 3, i % 4 < 2, i % 4 < 2


def test_choice_has_no_longer_chain_than_the_rules(choice):
    rng = random.Random(11)
    for p in PRODUCTS + list(_products(rng, 20000)):
        rule, pick = choice("shim_gemm", *p, ALL_ROOM)
        M, N, K = p[2:5]
        assert _chain(pick, M, N, K) <= _chain32(rule, M, N, K), p
    streamk = 0
    for c in _convs(rng, 20000):
        rule, pick = choice("shim_conv", *c, ALL_ROOM)
        assert _chain(pick, *c[:3]) <= _chain32(rule, *c[:3]), c
        streamk += rule.streamk and not pick.streamk
    assert streamk >= 50  # the stream-K rule's own regime is among them


def test_choice_takes_stream_k_only_with_tiles_for_half_the_chip(choice):
    """(a tile's last contributor adds the others' partial tiles in turn)"""
    for c in [(192, 40, 42336, 1, 1, 1), (49, 192, 50176, 1, 1, 1)] + list(_convs(random.Random(14), 20000)):
        _, pick = choice("shim_conv", *c, ALL_ROOM)
        assert not pick.streamk or -(-c[0] // 128) * -(-c[1] // 128) >= 128, c


def test_choice_at_less_workspace(choice):
    """A workspace of just what the choice asks for gives the same choice as a
    larger one; with less, the choice is neither predicted slower nor longer in
    its chain than what the rule runs there."""
    rng = random.Random(12)

    def check(fn, args, M, N, K, factors):
        _, full = choice(fn, *args, ALL_ROOM)
        if not full.streamk:
            need = full.splits * M * N * 4 if full.splits > 1 else 0
            _, same = choice(fn, *args, need)
            assert [getattr(same, n) for n, _ in _Pick._fields_] == [getattr(full, n) for n, _ in _Pick._fields_], args
        for f in factors:
            rule, pick = choice(fn, *args, int(f * M * N * 4))
            assert _chain(pick, M, N, K) <= _chain32(rule, M, N, K), (args, f)
            need = full.splits * M * N * 4 if full.splits > 1 else 0
            if rule.us >= 0 and pick.us >= 0 and (full.streamk or int(f * M * N * 4) < need):
                assert pick.us <= rule.us * (1 + 1e-6), (args, f)

    for p in PRODUCTS + list(_products(rng, 8000)):
        check("shim_gemm", p, *p[2:5], (0, rng.randint(2, 16)))
    for c in _convs(rng, 8000):
        check("shim_conv", c, *c[:3], (0, rng.randint(2, 16)))


@pytest.mark.parametrize("n,h,cin,k,cout,config,splits", [
    (1, 14, 129, 3, 130, "conv_64x64x32_w2x2_v11_dma2", 5), (1, 14, 132, 3, 130, "conv_64x64x32_w2x2_v41_dma2", 5),
    (2, 21, 3, 7, 30, "conv_64x64x16_w2x2_v11", 3), (1, 14, 515, 1, 130, "gemm_64x64x32_w2x2_nn_v11_dma2", 5)])
def test_measured_split_of_odd_channels_gets_its_workspace(pk, choice, n, h, cin, k, cout, config, splits):
    """The workspace query asks for the split that the search recorded for a
    convolution whose channels are no multiples of four."""
    lib, M = choice.lib, n * h * h
    lib.pk_conv2d_workspace_bytes_for.argtypes = pk.binding.SIGNATURES["pk_conv2d_workspace_bytes_for"][1]
    lib.pk_conv2d_workspace_bytes_for.restype = ctypes.c_size_t
    args = [None, n, h, h, cin, None, k, k, cout, 1, 1] + [k // 2] * 4
    assert lib.pk_conv2d_workspace_bytes_for(*args) != splits * M * cout * 4
    try:
        assert lib.shim_record(2 if k == 1 else 1, *map(ctypes.c_int64, (M, cout, k * k * cin)), k, 1, config.encode(), splits)
        assert lib.pk_conv2d_workspace_bytes_for(*args) == splits * M * cout * 4
    finally:
        lib.pk_tune_reset()


def test_workspace_query_for_the_operands_at_hand(pk, choice):
    """Operands aligned to 4 bytes only, or inside wider rows, get the workspace
    of the choice made for them, not of the aligned operands' one; a
    convolution's plain query holds every alignment's."""
    lib, rng = pk.load(), random.Random(13)
    differ = 0
    for i in range(3000):
        ta, tb, M, N, K, _ = next(_products(rng, 1))
        M, N, K = max(4, M // 4 * 4), max(4, N // 4 * 4), max(4, K // 4 * 4)
        _, pick = choice("shim_gemm", ta, tb, M, N, K, 0, ALL_ROOM)
        need = pick.splits * M * N * 4 if pick.splits > 1 else 0
        lda, ldb = (M if ta else K), (K if tb else N)
        sizes = [b"NT"[ta:ta + 1], b"NT"[tb:tb + 1], M, N, K]
        assert lib.pk_sgemm_workspace_bytes_for(*sizes, None, lda + 3, None, ldb, N) == need, sizes
        assert lib.pk_sgemm_workspace_bytes_for(*sizes, 4, lda, None, ldb, N) == need, sizes
        aligned = pk.binding.sgemm_workspace_bytes(bool(ta), bool(tb), M, N, K)
        assert lib.pk_sgemm_workspace_bytes_for(*sizes, None, lda, None, ldb, N) == aligned
        differ += aligned < need
    assert differ > 50
    differ = 0
    for i in range(3000):
        n, h, cin, cout, k = rng.randint(1, 32), _log(rng, 7, 100), 4 * _log(rng, 5, 200), 4 * _log(rng, 2, 200), rng.choice([3, 5])
        if k * k * cin < 500:  # (a direct form may take those)
            continue
        size, pads = [h, h, cin], [k // 2] * 4
        plain = pk.conv2d_workspace_bytes(n, h, h, cin, k, k, cout, 1, 1, *pads)
        for x, f, v in ((4, None, 0), (4, 4, 0), (None, 4, 1)):
            need = lib.pk_conv2d_workspace_bytes_for(x, n, *size, f, k, k, cout, 1, 1, *pads)
            _, pick = choice("shim_conv", n * h * h, cout, k * k * cin, v, 0, 1, ALL_ROOM)
            assert need == (pick.splits * n * h * h * cout * 4 if pick.splits > 1 else 0), (n, h, cin, cout, k)
            aligned = lib.pk_conv2d_workspace_bytes_for(None, n, *size, None, k, k, cout, 1, 1, *pads)
            assert plain >= max(need, aligned)
            differ += aligned < need
    assert differ > 50


@pytest.mark.parametrize("m,form,threads,channels", [(2, 0, 256, 32), (2, 1, 256, 64), (4, 0, 384, 32), (4, 1, 768, 64)])
def test_one_kernel_winograd_stays_within_a_grid(choice, m, form, threads, channels):
    """32 tiles to a work-group of `threads`: a launch holds fewer than 2^32
    work-items in x and at most 65535 blocks of channels in y."""
    def fits(T, cout):
        return choice.lib.shim_wino_fused_fits(m, form, ctypes.c_int64(T), ctypes.c_int64(cout))

    most = ((1 << 32) - 1) // threads * 32
    assert fits(1, 1) and fits(most, 65535 * channels)
    assert not fits(most + 1, 1) and not fits(1, 65535 * channels + 1)


# tiles, channels in and out, whether one kernel was measured faster than the three
@pytest.mark.parametrize("m,T,cin,cout,one", [
    (4, 960, 72, 638, False), (4, 4212, 80, 117, False), (4, 192, 96, 918, False), (2, 2809, 732, 20, False),
    (2, 2420, 540, 48, False),
    (2, 3136, 64, 64, True), (2, 25088, 256, 256, True), (4, 6272, 64, 64, True)])
def test_one_kernel_winograd_only_where_faster(choice, m, T, cin, cout, one):
    form = choice.lib.shim_wino_form(m, *map(ctypes.c_int64, (T, cin, cout)))
    assert (form >= 0) == one


# n, h, w, cin, window, cout, stride; the tile with its groups and the least split
# that were measured slower than the rule's
@pytest.mark.parametrize("n,h,w,cin,k,cout,s,tile,splits", [
    (9, 116, 116, 256, 3, 192, 2, (64, 64, 32, 4), 1), (8, 51, 51, 196, 5, 144, 1, (64, 64, 32, 4), 1),
    (5, 109, 109, 136, 5, 56, 1, (64, 64, 32, 4), 1),
    (25, 29, 29, 72, 3, 64, 1, (32, 64, 32, 1), 1), (6, 20, 13, 32, 3, 704, 1, (32, 64, 32, 1), 1),
    (21, 10, 10, 28, 7, 128, 2, (32, 64, 32, 1), 1), (14, 20, 31, 32, 5, 80, 2, (64, 64, 16, 1), 12),
    (4, 12, 12, 112, 3, 600, 1, (64, 64, 16, 1), 8), (5, 10, 10, 108, 3, 912, 2, (64, 64, 16, 1), 16)])
def test_conv_choice_avoids_what_was_measured_slower(choice, n, h, w, cin, k, cout, s, tile, splits):
    _, pick = choice("shim_conv", n * -(-h // s) * -(-w // s), cout, k * k * cin, 1, 1, 1, ALL_ROOM)
    assert (pick.bm, pick.bn, pick.bk, pick.kg) != tile or pick.splits < splits


@pytest.mark.parametrize("M,N,K", [(15975, 857, 51), (29403, 971, 64), (93636, 459, 64), (15975, 857, 128), (14336, 900, 135)])
def test_large_tiles_need_a_reduction(choice, M, N, K):
    """256 x 256 tiles were measured up to 1.4 times slower there."""
    _, pick = choice("shim_gemm", 0, 0, M, N, K, 0, ALL_ROOM)
    assert pick.bm * pick.bn < 256 * 256


@pytest.mark.parametrize("ta,tb,M,N,K", [(1, 0, 544, 3816, 1826), (0, 0, 968, 2656, 632)])
def test_gemm_choice_avoids_what_was_measured_slower(choice, ta, tb, M, N, K):
    _, pick = choice("shim_gemm", ta, tb, M, N, K, 1, ALL_ROOM)
    assert (pick.bm, pick.bn) != (128, 96)
