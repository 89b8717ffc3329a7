"""The few-row kernel (fewer than 256 rows at G >= 128 or per channel): its forms
of 16 and 32 rows by 32 or 64 columns (SHAPES) and of 64 rows by 64 columns
(FORMS_64), at the edges of their rows and columns, with fewer stages than
waves, with scale rows of every alignment (K/G a multiple of 8 or not),
sub-group partials and a partial last stage per channel.

  * Y within the tolerance of the oracle in full, the same bits on both weight
    layouts, through the workspace entry point when it picks the same kernel,
    and from the debug form;
  * the exact group sums of a row window against the oracle;
  * one row with the quantizer in the prologue (tiled weights): Y and the work
    buffers equal the quantizer followed by the GEMM, bit for bit.
"""
import ctypes

import numpy as np
import pytest

from parity import check_tolerance, dev, host, log
from paper_2606_08761_amd import workloads as wl

pytestmark = pytest.mark.gpu


def pk():
    import paper_2606_08761_amd as m
    return m


# (M, N, K, G): the 16- and 32-row forms at the first and last row counts (16 /
# 17, 32 / 33, 64 / 65, 255); one column, one past a tile, an odd count of 32-column tiles;
# one stage (seven idle waves), 9 stages, 26 and 27 groups (not a multiple of
# 8); more column tiles than eight XCDs take evenly; G = 256, 512, 1024; per
# channel with whole and partial last stages
SHAPES = [(1, 33, 128, 128), (15, 1, 1152, 128), (16, 1000, 3328, 128), (17, 65, 1024, 128), (31, 8200, 256, 128),
          (32, 8224, 1152, 128), (33, 1000, 3328, 128), (64, 520, 128, 128), (65, 2080, 1024, 128), (96, 16500, 256, 128),
          (129, 4100, 640, 128), (255, 1056, 3456, 128), (200, 8200, 512, 128),
          (16, 96, 2048, 256), (48, 1000, 2048, 512), (130, 520, 3072, 1024),
          (9, 100, 96, 96), (16, 520, 4000, 4000), (32, 1000, 8192, 8192), (40, 65, 4000, 4000), (250, 2000, 1120, 1120)]


FORMS = ("16x32", "32x32", "32x64", "32x64 four waves", "64x64", "64x64 four waves")


def form(M, N, K, G):
    """The form that the library chooses (no entry point tells: its own function, by its C++ name)."""
    f = pk().lib()._ZN5apex412rows_form_ofEllll
    f.argtypes = [ctypes.c_int64] * 4
    return FORMS[f(M, N, K, G)]


# the form of each of SHAPES on 256 CUs, beside its sizes
EXPECT = {(15, 1, 1152, 128): 0, (16, 1000, 3328, 128): 0, (17, 65, 1024, 128): 1, (31, 8200, 256, 128): 2,
          (33, 1000, 3328, 128): 2, (65, 2080, 1024, 128): 2, (96, 16500, 256, 128): 3, (129, 4100, 640, 128): 3,
          (200, 8200, 512, 128): 3, (32, 1000, 8192, 8192): 1, (250, 2000, 1120, 1120): 2}


@pytest.mark.parametrize("M,N,K,G", SHAPES)
def test_rows(O, M, N, K, G):
    import torch
    m = pk()
    plan, plan_ws = (m.apex4_w4a4_gemm_plan(e, M, N, K, G) for e in ("gemm", "gemm_ws"))
    log(f"rows M={M} N={N} K={K} G={G}: {plan} {form(M, N, K, G)}, with a workspace {plan_ws}")
    assert M == 1 or plan == ("decode", 1)
    if (M, N, K, G) in EXPECT:
        assert form(M, N, K, G) == FORMS[EXPECT[M, N, K, G]]
    r = np.random.default_rng(M * 31 + N * 7 + K + G)
    Aq, Wq = wl.random_codes(r, M, K), wl.random_codes(r, N, K)
    sa, sw = wl.random_scales(r, M, K // G), wl.random_scales(r, N, K // G)
    d = [dev(a) for a in (Aq, sa, Wq, sw)]
    need = m.apex4_w4a4_gemm_workspace_size(M, N, K, G)
    ws = torch.empty((max(need, 16),), dtype=torch.uint8, device="cuda")
    Y = m.apex4_w4a4_gemm(*d, G)
    Yw = m.apex4_w4a4_gemm_ws(*d, G, ws)
    m0, mr = M // 3, min(7, M - M // 3)
    Yd, P = m.apex4_w4a4_gemm_debug(*d, G, m0, mr)
    P2 = m.apex4_w4a4_gemm_groupsums(d[0], d[2], G, m0, mr)
    out = [Yd]
    if G >= 128 and M > 1:  # one row: the dot-product kernel on row-major weights
        Wt = m.apex4_tile_weights(d[2])
        out.append(m.apex4_w4a4_gemm_tiled(d[0], d[1], Wt, d[3], G))
        out.append(m.apex4_w4a4_gemm_debug(d[0], d[1], Wt, d[3], G, m0, mr, flags=m.APEX4_DEBUG_W_TILED)[0])
    elif G >= 128:
        check_tolerance(host(m.apex4_w4a4_gemm_tiled(d[0], d[1], m.apex4_tile_weights(d[2]), d[3], G)),
                        O.gemm_rows(Aq, sa, Wq, sw, K, G), f"rows tiled {M}x{N}x{K} G{G}")
    if plan_ws[0] == plan[0]:
        out.append(Yw)
    torch.cuda.synchronize()
    assert all(torch.equal(y, Y) for y in out)
    P_o = O.groupsums(Aq, Wq, K, G, m0, mr)
    assert np.array_equal(host(P), P_o) and np.array_equal(host(P2), P_o)
    y = O.gemm_rows(Aq, sa, Wq, sw, K, G)
    check_tolerance(host(Y), y, f"rows {M}x{N}x{K} G{G}")
    check_tolerance(host(Yw), y, f"rows with a workspace {M}x{N}x{K} G{G}")


# (M, N, K, G, waves): 64 rows by 64 columns, in workgroups of eight and of four
# waves; one row past a block, two blocks, the last of four; ragged columns (an
# odd count of 32-column tiles); a stage, a group and the row to a scale, a
# partial last stage; K/G a multiple of 8 and not
FORMS_64 = [(65, 8190, 8192, 128, 8), (72, 8190, 8192, 128, 8), (128, 8150, 8320, 128, 8), (255, 16390, 4096, 128, 4),
            (128, 33000, 4224, 128, 4), (72, 8190, 2048, 256, 8), (128, 20470, 8192, 256, 4), (100, 8190, 8192, 1024, 8),
            (72, 8190, 4000, 4000, 8), (128, 8150, 2016, 2016, 8), (200, 4096, 4096, 4096, 8), (182, 35473, 1856, 1856, 4)]


@pytest.mark.parametrize("M,N,K,G,waves", FORMS_64)
def test_rows_64(O, M, N, K, G, waves):
    """Y on sampled rows (both ends of every block) against the oracle, on both
    weight layouts and from the debug form, and the exact group sums of a window
    across the first block's end."""
    import torch
    m = pk()
    assert m.apex4_w4a4_gemm_plan("gemm", M, N, K, G) == ("decode", 1)
    assert form(M, N, K, G) == FORMS[4 if waves == 8 else 5]
    log(f"rows 64x64 M={M} N={N} K={K} G={G}")
    r = np.random.default_rng(M * 31 + N * 7 + K + G)
    Aq, Wq = wl.random_codes(r, M, K), wl.random_codes(r, N, K)
    sa, sw = wl.random_scales(r, M, K // G), wl.random_scales(r, N, K // G)
    d = [dev(a) for a in (Aq, sa, Wq, sw)]
    Wt = m.apex4_tile_weights(d[2])
    m0, mr = 61, min(8, M - 61)
    Y = m.apex4_w4a4_gemm(*d, G)
    Yt = m.apex4_w4a4_gemm_tiled(d[0], d[1], Wt, d[3], G)
    Yd, P = m.apex4_w4a4_gemm_debug(*d, G, m0, mr)
    Ydt, Pt = m.apex4_w4a4_gemm_debug(d[0], d[1], Wt, d[3], G, m0, mr, flags=m.APEX4_DEBUG_W_TILED)
    P2 = m.apex4_w4a4_gemm_groupsums(d[0], d[2], G, m0, mr)
    torch.cuda.synchronize()
    assert torch.equal(Yt, Y) and torch.equal(Yd, Y) and torch.equal(Ydt, Y)
    P_o = O.groupsums(Aq, Wq, K, G, m0, mr)
    assert all(np.array_equal(host(p), P_o) for p in (P, Pt, P2))
    rows = np.unique([i for b in range(0, M, 64) for i in (b, b + 15, b + 16, b + 31, b + 32, b + 63) if i < M] + [M - 1])
    check_tolerance(host(Y)[rows], O.gemm_rows(Aq, sa, Wq, sw, K, G, rows), f"rows 64x64 {M}x{N}x{K} G{G}")


@pytest.mark.parametrize("N,K,G", [(1, 256, 128), (33, 3328, 128), (1000, 5120, 256), (9000, 4096, 512), (64, 40960, 128)])
def test_rows_fused_one_row(O, N, K, G):
    import torch
    m = pk()
    T = m.APEX4_DEBUG_W_TILED
    assert m.apex4_w4a4_gemm_plan("linear", 1, N, K, G, T) == ("fused", 1)
    x, w = wl.activations(wl.rng_for("decode", 61, N + K), 1, K), wl.weights(wl.rng_for("decode", 62, N + K), N, K)
    Wq, sw = m.apex4_quantize_act(dev(w), G)
    Wt = m.apex4_tile_weights(Wq)
    Aq, sa = m.apex4_quantize_act(dev(x), G)
    Aw = torch.full_like(Aq, 0xAB)
    sw_ = torch.full_like(sa, float("nan"))
    Y = m.apex4_w4a4_linear_tiled(dev(x), Wt, sw, G, A_q_work=Aw, s_a_work=sw_)
    Yg = m.apex4_w4a4_gemm_tiled(Aq, sa, Wt, sw, G)
    Yd, _, _, P = m.apex4_w4a4_linear_debug(dev(x), Wt, sw, G, flags=T)
    torch.cuda.synchronize()
    assert torch.equal(Y, Yg) and torch.equal(Yd, Y)
    assert torch.equal(Aw, Aq) and torch.equal(sw_.view(torch.int16), sa.view(torch.int16))
    Aq_o, sa_o = O.quantize(x, G)
    Wq_o, sw_o = O.quantize(w, G)
    assert np.array_equal(host(P), O.groupsums(Aq_o, Wq_o, K, G))
    check_tolerance(host(Y), O.gemm_rows(Aq_o, sa_o, Wq_o, sw_o, K, G), f"rows fused N={N} K={K} G={G}")


def formula(O, Aq, sa, Wq, sw, K, G):
    """Y = sum_g s_a s_w P in binary64 with IEEE infinities and NaN."""
    P = O.groupsums(Aq, Wq, K, G).astype(np.float64)
    with np.errstate(invalid="ignore"):
        return (sa.astype(np.float64)[:, None, :] * (sw.astype(np.float64)[None] * P)).sum(axis=2)


# (M, N, K, G), K/128 not a multiple of the waves (past K they have no stage):
# 16, 32 and 64 rows a workgroup, fewer stages than waves, per channel with a
# partial last stage
DEAD = [(1, 33, 1152, 128), (16, 100, 1152, 128), (20, 100, 384, 128), (40, 200, 1152, 128), (72, 8192, 1152, 128),
        (16, 100, 1184, 1184), (40, 200, 1184, 1184)]


@pytest.mark.parametrize("M,N,K,G", DEAD)
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_rows_non_finite_scale(O, M, N, K, G, value):
    """A non-finite activation scale gives what the formula gives, and only in
    its own row: no wave multiplies it with a weight scale that is not there."""
    m = pk()
    r = np.random.default_rng(M + N + K + G)
    Aq, Wq = wl.random_codes(r, M, K), wl.random_codes(r, N, K)
    sa, sw = wl.random_scales(r, M, K // G), wl.random_scales(r, N, K // G)
    sa[M // 2, -1] = value   # the last group: the one that waves past K would read
    log(f"rows scale {value} M={M} N={N} K={K} G={G}: {m.apex4_w4a4_gemm_plan('gemm', M, N, K, G)}")
    d = [dev(a) for a in (Aq, sa, Wq, sw)]
    outs = [m.apex4_w4a4_gemm_tiled(d[0], d[1], m.apex4_tile_weights(d[2]), d[3], G)]
    if M > 1:  # one row on row-major weights is the dot-product kernel, which scales parts of a group
        outs.append(m.apex4_w4a4_gemm(*d, G))
    y = formula(O, Aq, sa, Wq, sw, K, G)
    bad = np.arange(M) == M // 2
    assert not np.isfinite(y[bad]).any()
    for Y in outs:
        Y = host(Y)
        check_tolerance(Y[~bad], y[~bad]) if M > 1 else None
        assert np.array_equal(Y[bad], y[bad].astype(np.float16), equal_nan=True)


# groups of several 128-wide stages at 33 rows and more: 32- and 64-row forms of
# eight and of four waves, group counts that the waves share evenly and not
WHOLE = [(33, 200, 2048, 256), (72, 1000, 5120, 512), (40, 8200, 9216, 1024), (200, 4096, 8192, 512), (255, 2000, 4096, 256),
         (64, 520, 3072, 1024), (130, 1000, 28672, 1024), (72, 8192, 2048, 256), (128, 20470, 8192, 256)]


@pytest.mark.parametrize("M,N,K,G", WHOLE)
def test_rows_group_sums_whole(O, M, N, K, G):
    """A group's sum is added up in integers before it meets its scales, also
    where several 128-wide stages make up a group.

      * Opposite halves: every group's first half sums to several thousand and
        its second half takes nearly all of it away again.  Scaled by halves in
        binary32, the two would leave errors of 2^-24 of the halves, hundreds
        of times 2^-24 of the result (2 to 20 % of the roundings below differ
        then); whole, Y is the binary16 rounding of the exact value but where
        that lies within about 2^-24 (K/G + 8) of a tie: 2^-12 (K/G + 8) of
        the results at most, and errors add up in a walk, so far fewer.
      * An infinite activation scale gives infinities by the sign of the whole
        group's sum."""
    m = pk()
    plan = m.apex4_w4a4_gemm_plan("gemm", M, N, K, G)
    log(f"rows whole groups M={M} N={N} K={K} G={G}: {plan}")
    assert plan[0] == "decode"
    r = np.random.default_rng(M + N + K + G)
    rows = np.unique([0, 31, 32, M // 2, min(63, M - 1), min(64, M - 1), M - 1])
    half = G // 2
    a = r.integers(4, 8, (M, K // G, G), dtype=np.int8)
    w = r.integers(4, 8, (N, K // G, G), dtype=np.int8)
    a[:, :, half:] = -a[:, :, :half]
    w[:, :, half:] = w[:, :, :half]
    k = r.integers(0, half, (M, K // G, 1))
    np.put_along_axis(a, k, np.take_along_axis(a, k, 2) - np.int8(1), 2)   # one code of each group differs
    pack = lambda v: ((v[..., 0::2] & 0xF) | ((v[..., 1::2] & 0xF) << 4)).astype(np.uint8).reshape(len(v), K // 2)
    Aq, Wq = pack(a), pack(w)
    del a, w
    sa, sw = wl.random_scales(r, M, K // G), wl.random_scales(r, N, K // G)
    y = formula(O, Aq[rows], sa[rows], Wq, sw, K, G)
    d = [dev(v) for v in (Aq, sa, Wq, sw)]
    Y = host(m.apex4_w4a4_gemm(*d, G))[rows]
    check_tolerance(Y, y, f"whole groups {M}x{N}x{K} G{G}")
    wrong = (Y != y.astype(np.float16)).mean()
    log(f"  roundings that differ: {wrong:.2e}")
    assert wrong < 2e-3

    Aq, Wq = wl.random_codes(r, M, K), wl.random_codes(r, N, K)
    sa[M // 2, 0] = np.inf
    y = formula(O, Aq[[M // 2]], sa[[M // 2]], Wq, sw, K, G)
    Y = host(m.apex4_w4a4_gemm(dev(Aq), dev(sa), dev(Wq), d[3], G))
    assert np.array_equal(Y[[M // 2]], y.astype(np.float16), equal_nan=True)
    assert np.isfinite(np.delete(Y, M // 2, 0)).all()
