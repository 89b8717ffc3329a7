"""The kernel choice of the GEMM, on the CPU (no GPU needed: without one the
library plans for 256 compute units).  The choice has no entry point that works
without a device, so the library's own functions are called by their C++ names.

Over seeded shapes of every group size:
  * a workspace is asked for exactly where the chosen kernel uses one, and
    where none is, the choice is the one without a workspace;
  * the few-row kernel is only chosen for shapes that it takes, and loads
    weights past the caches (nontemporal) only where they are tiled and read once.
"""
import ctypes
import random

import pytest

I = ctypes.c_int64
GEMV, DECODE, TILE64, TILE128, PINGPONG, DECODE_SPLIT = 1, 3, 4, 5, 6, 7


class Plan(ctypes.Structure):
    _fields_ = [("kernel", ctypes.c_int), ("splits", ctypes.c_int)]


@pytest.fixture(scope="module")
def lib():
    import paper_2606_08761_amd as m
    L = m.lib()

    def fn(name, restype, *more):
        f = getattr(L, name)
        f.restype, f.argtypes = restype, [I] * 4 + list(more)
        return f
    b = ctypes.c_bool
    plan = fn("_ZN5apex49plan_gemmEllllbbb", Plan, b, b, b)
    return {"plan": lambda M, N, K, G, split, wt=False: (lambda p: (p.kernel, p.splits))(plan(M, N, K, G, split, False, wt)),
            "workspace": fn("_ZN5apex422splitk_workspace_bytesEllll", I),
            "rows_fits": fn("_ZN5apex49rows_fitsEllll", b),
            "fused": fn("_ZN5apex415rows_fused_fitsEllll", b),
            "nontemporal": _nontemporal(L)}


def _nontemporal(L):
    f = L._ZN5apex416rows_nontemporalElllb
    f.restype, f.argtypes = ctypes.c_bool, [I] * 3 + [ctypes.c_bool]
    return f


def shapes(n, seed):
    r = random.Random(seed)
    while n:
        G = r.choice([32, 64, 128, 256, 512, 1024, 0])
        M, N = round(2 ** (11 * r.random())), round(2 ** (16 * r.random()))
        K = 32 * r.randint(1, 2048) if G in (0, 32) else G * r.randint(1, 65536 // G)
        yield M, N, K, G or K
        n -= 1


def test_workspace_is_what_the_kernel_uses(lib):
    kernels = set()
    for M, N, K, G in shapes(20000, 1):
        kernel, S = lib["plan"](M, N, K, G, True)
        need = lib["workspace"](M, N, K, G)
        at = (M, N, K, G, kernel, S, need)
        kernels.add((kernel, S > 1))
        if S > 1:
            assert kernel in (TILE64, PINGPONG) and need == S * M * N * 4, at
        elif kernel == DECODE_SPLIT:
            assert need > 0, at
        else:
            assert need == 0 and lib["plan"](M, N, K, G, False) == (kernel, 1), at
    assert kernels == {(GEMV, False), (DECODE, False), (DECODE_SPLIT, False), (TILE64, False), (TILE64, True),
                       (TILE128, False), (PINGPONG, False), (PINGPONG, True)}


def test_few_row_kernel_takes_what_it_is_chosen_for(lib):
    for M, N, K, G in shapes(20000, 2):
        for wt in (False, True) if G >= 128 else (False,):
            for split in (False, True):
                kernel, _ = lib["plan"](M, N, K, G, split, wt)
                if kernel == DECODE and G >= 128:
                    assert lib["rows_fits"](M, N, K, G), (M, N, K, G, wt, split)
                if kernel == DECODE:
                    assert M < 256, (M, N, K, G)


def test_few_row_kernel_streams_tiled_weights_only(lib):
    f = lib["nontemporal"]
    for M, N, K, G in shapes(20000, 3):
        assert not f(M, N, K, False), (M, N, K)
        assert f(M, N, K, True) == (M <= 32 and N * (K // 2) >= 16 << 20), (M, N, K)


def test_fused_row_is_bounded(lib):
    """One row on tiled weights: every workgroup quantizes all of x, so the fused
    form ends where a separate quantizer is the faster way (long K; at G = 512
    many columns), and at the groups that a wave holds."""
    f = lib["fused"]
    for G in (128, 256, 512):
        assert f(1, 8192, 8192, G) and f(1, 16384, 16384, G) and f(1, 64, 40960, G)
        assert not f(1, 8192, 16384 + G, G) and not f(1, 2048, 57344, G) and not f(2, 8192, 8192, G)
        assert f(1, 57344, 8192, G) == (G < 512)
    assert not f(1, 8192, 8192, 1024) and not f(1, 512, 512, 512)
    for _, N, K, G in shapes(20000, 4):
        if f(1, N, K, G):
            assert G in (128, 256, 512) and G < K and (K <= 16384 or N * K <= 33 << 18), (N, K, G)


# (M, N, K, stream-K or not) at G = 128 on 256 CUs, on both sides of each line
SPLIT_LINES = [(16, 2048, 16384, True), (16, 2560, 24576, False), (9, 2560, 28672, True), (8, 2560, 28672, False),
               (8, 2560, 32768, True), (32, 3072, 32768, True), (32, 3584, 32768, False), (2, 3584, 57344, True),
               (32, 8192, 57344, False), (2, 9216, 24576, True), (16, 10240, 24576, False), (16, 10240, 28672, True),
               (17, 10240, 28672, False), (9, 17408, 28672, True), (8, 17408, 28672, False), (16, 12288, 57344, False)]


def test_stream_k_where_it_pays(lib):
    for M, N, K, split in SPLIT_LINES:
        for wt in (False, True):
            if M > 2 or not wt:  # two rows on tiled weights: the dot-product kernel
                assert (lib["plan"](M, N, K, 128, True, wt) == (DECODE_SPLIT, 1)) == split, (M, N, K, wt)
