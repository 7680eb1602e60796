"""GPU library vs the oracle, element by element (pair sets), on seeded inputs.

Integer-valued inputs must give identical pair sets; real-valued inputs must
agree outside the boundary band 1e-3 * |threshold| (those pairs are excluded
and counted).  Cases cover every kernel variant (d picks the k-step variant;
d > 256 takes the K-streamed kernel), ragged n against the tile sizes,
unaligned rows, both metrics, both modes, edge cases, and the full-size
workloads on sampled rows.
"""
import sys

import numpy as np
import pytest

import oracle
import workloads
from gpu_util import compare, gpu_join, keys, sorted_pairs, to_device
from pins import values

pytestmark = pytest.mark.gpu


def say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2006_12608_amd  # noqa: F401  (fails loudly when libsj.so is missing)
    yield
    torch.cuda.synchronize()


def run_case(w, thr=None, two_pass=False, rows=None):
    thr = w.threshold if thr is None else thr
    Pd, Qd = to_device(w.P, w.dtype), to_device(w.Q, w.dtype)
    if w.self_join:
        Qd = Pd
    say(w.name, w.metric, w.dtype, w.n_p, w.n_q, w.d, thr, "two_pass" if two_pass else "single")
    g = sorted_pairs(gpu_join(w.metric, Pd, Qd, thr, two_pass=two_pass))
    band = 1e-3 * abs(thr) if w.real_valued else 0.0
    ref = oracle.join(w.metric, w.dtype, w.P, w.Q, thr, band=band, rows=rows)
    if rows is not None:
        g = g[np.isin(g[:, 0], np.asarray(rows))]
    return compare(g, ref, w.real_valued), g, ref


# ------------------------------------------------------- the five workloads

@pytest.mark.parametrize("k,n", [("ip_f16_2048x64", None), ("ip_bf16_65536x128", 2048),
                                 ("cos_f16_262144x256", 2048), ("l2_i8_1048576x64", 4096),
                                 ("ip_bf16_clustered_131072x1024", 1024)])
@pytest.mark.parametrize("two_pass", [False, True])
def test_workload_reduced(k, n, two_pass):
    w = workloads.make_config(k, n=n)
    info, g, ref = run_case(w, two_pass=two_pass)
    if w.planted.size:
        assert set(map(tuple, w.planted.tolist())) <= set(map(tuple, g.astype(np.int64).tolist()))
    if w.real_valued:
        say("band", info)


def test_true_self_join():
    w = workloads.make_config("ip_f16_2048x64", self_join=True)
    _, g, _ = run_case(w)
    s = set(map(tuple, g.tolist()))
    assert s == {(j, i) for (i, j) in s}


# ------------------------------------------------------ random shapes

DIMS = [1, 7, 16, 33, 64, 65, 100, 128, 200, 256, 257, 600, 1024]
SHAPES = [(300, 517), (70, 1), (1030, 129), (513, 64)]


def _case(seed, dtype, d, shape, metric):
    n_p, n_q = shape
    lo, hi = (-8, 8) if dtype != "i8" else (-128, 127)
    if dtype != "i8" and metric == "l2":
        lo, hi = -20, 20
    w = workloads.random_case(seed, n_p, n_q, d, dtype, lo=lo, hi=hi, metric=metric)
    x = values(dtype, w.P).astype(np.int64)
    y = values(dtype, w.Q).astype(np.int64)
    if metric == "ip":
        S = x @ y.T
        q = 0.5 if seed % 3 == 0 else 0.99
        w.threshold = float(np.quantile(S, q, method="nearest"))
    else:
        D = (x * x).sum(1)[:, None] + (y * y).sum(1)[None, :] - 2 * (x @ y.T)
        q = 0.5 if seed % 3 == 0 else 0.01
        w.threshold = float(np.quantile(D, q, method="nearest"))
    return w


@pytest.mark.parametrize("metric", ["ip", "l2"])
@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
@pytest.mark.parametrize("d", DIMS)
def test_random_shapes(d, dtype, metric):
    seed = 100 + DIMS.index(d) * 7 + ["f16", "bf16", "i8"].index(dtype) * 3 + (metric == "l2")
    shape = SHAPES[seed % len(SHAPES)]
    w = _case(seed, dtype, d, shape, metric)
    run_case(w, two_pass=(seed % 2 == 1))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("metric", ["ip", "l2"])
def test_real_valued_band(dtype, metric):
    w = workloads.random_case(7, 700, 900, 96, dtype, real=True, metric=metric)
    x, y = values(dtype, w.P), values(dtype, w.Q)
    if metric == "ip":
        thr = float(np.quantile(x @ y.T, 0.995))
    else:
        D = (x * x).sum(1)[:, None] + (y * y).sum(1)[None, :] - 2 * (x @ y.T)
        thr = float(np.quantile(D, 0.01))
    info, _, _ = run_case(w, thr=thr)
    say("band", info)


@pytest.mark.parametrize("dtype,metric", [("f16", "ip"), ("bf16", "l2")])
def test_real_valued_band_streamed_two_pass(dtype, metric):
    """Real-valued rows long enough for the K-streamed kernel, count-then-emit
    (the first pass's match bits): equal to the oracle outside the band."""
    w = workloads.random_case(8, 520, 610, 400, dtype, real=True, metric=metric)
    x, y = values(dtype, w.P), values(dtype, w.Q)
    if metric == "ip":
        thr = float(np.quantile(x @ y.T, 0.99))
    else:
        D = (x * x).sum(1)[:, None] + (y * y).sum(1)[None, :] - 2 * (x @ y.T)
        thr = float(np.quantile(D, 0.01))
    info, _, _ = run_case(w, thr=thr, two_pass=True)
    say("band", info)


# ------------------------------------------------------- protocol / edges

def test_two_pass_is_deterministic_and_equals_single():
    import torch
    w = workloads.make_config("ip_bf16_clustered_131072x1024", n=1024)
    Pd, Qd = to_device(w.P, "bf16"), to_device(w.Q, "bf16")
    say("two-pass determinism", w.name)
    a = gpu_join("ip", Pd, Qd, w.threshold, two_pass=True)
    b = gpu_join("ip", Pd, Qd, w.threshold, two_pass=True)
    assert torch.equal(a, b)            # same order, not only the same set
    c = gpu_join("ip", Pd, Qd, w.threshold, two_pass=False)
    assert np.array_equal(sorted_pairs(a), sorted_pairs(c))


def test_overflow_reports_exact_total():
    import torch
    import paper_2006_12608_amd as sj
    w = workloads.make_config("ip_f16_2048x64")
    Pd, Qd = to_device(w.P, "f16"), to_device(w.Q, "f16")
    total = oracle.count("ip", "f16", w.P, w.Q, w.threshold)
    say("overflow", total)
    assert sj.count(Pd, Qd, w.threshold) == total
    for two_pass in (False, True):
        for cap in (0, total - 1):
            out = torch.empty((max(cap, 1), 2), dtype=torch.int32, device="cuda")
            with pytest.raises(sj.SjError) as e:
                sj.join_ip(Pd, Qd, w.threshold, cap=cap, out=out, two_pass=two_pass)
            assert e.value.status == sj.SJ_E_OVERFLOW and e.value.n_out == total
        out = torch.empty((total, 2), dtype=torch.int32, device="cuda")
        r = sj.join_ip(Pd, Qd, w.threshold, cap=total, out=out, two_pass=two_pass)
        assert r.shape[0] == total


@pytest.mark.parametrize("dtype", ["f16", "bf16", "i8"])
def test_extreme_thresholds(dtype):
    import paper_2006_12608_amd as sj
    w = workloads.random_case(3, 130, 70, 40, dtype)
    Pd, Qd = to_device(w.P, dtype), to_device(w.Q, dtype)
    say("extreme thresholds", dtype)
    for metric in ("ip", "l2"):
        f = sj.join_ip if metric == "ip" else sj.join_l2
        all_thr, none_thr = (-np.inf, np.inf) if metric == "ip" else (np.inf, -np.inf)
        assert f(Pd, Qd, all_thr).shape[0] == 130 * 70
        assert f(Pd, Qd, none_thr).shape[0] == 0
        big = 1e30 if metric == "ip" else -1.0
        assert f(Pd, Qd, big).shape[0] == 0
        huge = -1e30 if metric == "ip" else 1e30
        assert sj.count(Pd, Qd, huge, metric) == 130 * 70


@pytest.mark.parametrize("dtype,metric", [("i8", "l2"), ("i8", "ip"), ("f16", "ip"),
                                          ("bf16", "l2")])
def test_maximum_d(dtype, metric):
    """The longest rows the library takes (d = 32768 int8, 65536 fp16 / bf16:
    the K-streamed kernel over 256 or 1024 chunks of 128 bytes), 40 x 300 rows
    (ragged against the 256-row tiles), both modes.  int8 row 0 of P is all
    127, row 1 of P and rows 0 and 1 of Q all -128, and the thresholds include
    the largest squared distance int8 rows of this length can have (32768 *
    255^2 = 2130739200, inside int32: every pair matches, row pair (0, 0) as a
    tie) and the largest inner product (32768 * 128^2: row pairs (1, 0) and
    (1, 1) only)."""
    d = 32768 if dtype == "i8" else 65536
    lo, hi = (-128, 127) if dtype == "i8" else (-4, 4)
    rng = np.random.default_rng(5150 + 2 * (dtype == "i8") + (metric == "l2"))
    Pv = rng.integers(lo, hi + 1, size=(40, d))
    Qv = rng.integers(lo, hi + 1, size=(300, d))
    if dtype == "i8":
        Pv[0], Qv[0], Pv[1], Qv[1] = 127, -128, -128, -128
    x, y = Pv.astype(np.float64), Qv.astype(np.float64)   # sums stay below 2^53: exact
    if metric == "ip":
        thrs = [float(np.quantile(x @ y.T, 0.9, method="nearest"))]
        if dtype == "i8":
            thrs.append(float(32768 * 128 * 128))
    else:
        D = (x * x).sum(1)[:, None] + (y * y).sum(1)[None, :] - 2 * (x @ y.T)
        thrs = [float(np.quantile(D, 0.1, method="nearest"))]
        if dtype == "i8":
            thrs.append(float(32768 * 255 * 255))
    w = workloads.Workload(f"maxd_{dtype}_{d}", metric, dtype, workloads.encode(Pv, dtype),
                           workloads.encode(Qv, dtype), 0.0, np.zeros((0, 2), np.int64))
    for thr in thrs:
        for two_pass in (False, True):
            _, g, ref = run_case(w, thr=thr, two_pass=two_pass)
            if dtype == "i8" and thr == 32768 * 255 * 255:
                assert g.shape[0] == 40 * 300
            if dtype == "i8" and thr == 32768 * 128 * 128:
                assert g.tolist() == [[1, 0], [1, 1]]


@pytest.mark.parametrize("dtype,d", [("bf16", 600), ("f16", 1024), ("i8", 700)])
def test_streamed_dense_output(dtype, d):
    """The K-streamed kernel with every pair matching (each wave's staging
    buffer fills several times per output block) and with about half the pairs
    matching, in both modes, against the oracle."""
    import paper_2006_12608_amd as sj
    w = workloads.random_case(21, 300, 517, d, dtype, lo=-2, hi=2)
    Pd, Qd = to_device(w.P, dtype), to_device(w.Q, dtype)
    say("streamed dense", dtype, d)
    for two_pass in (False, True):
        allp = sorted_pairs(sj.join_ip(Pd, Qd, -np.inf, two_pass=two_pass))
        assert allp.shape[0] == 300 * 517
        assert np.array_equal(allp[:, 0], np.repeat(np.arange(300), 517))
        assert np.array_equal(allp[:, 1], np.tile(np.arange(517), 300))
    x = values(dtype, w.P).astype(np.int64)
    y = values(dtype, w.Q).astype(np.int64)
    w.threshold = float(np.quantile(x @ y.T, 0.5, method="nearest"))
    for two_pass in (False, True):
        run_case(w, two_pass=two_pass)


@pytest.mark.parametrize("dtype,d,metric", [("f16", 256, "ip"), ("bf16", 100, "l2"),
                                             ("i8", 64, "l2"), ("i8", 16, "ip")])
@pytest.mark.parametrize("n_p", [1, 64, 65, 200, 513, 1100])
def test_few_rows_against_many(dtype, d, metric, n_p):
    """Few rows of P against many of Q: one Q tile per workgroup and waves
    without rows (which only load tiles), all modes, integer inputs: the
    oracle's set, and count-then-emit's order whichever second pass runs."""
    import paper_2006_12608_amd as sj
    w = workloads.random_case(60 + n_p + d, n_p, 9001, d, dtype, lo=-3, hi=3, metric=metric)
    x, y = values(dtype, w.P).astype(np.int64), values(dtype, w.Q).astype(np.int64)
    s = x @ y.T
    if metric == "l2":
        s = (x * x).sum(1)[:, None] + (y * y).sum(1)[None, :] - 2 * s
    w.threshold = float(np.quantile(s, 0.99 if metric == "ip" else 0.01, method="nearest"))
    _, g, _ = run_case(w)
    _, h, _ = run_case(w, two_pass=True)
    assert np.array_equal(g, h)
    Pd, Qd = to_device(w.P, dtype), to_device(w.Q, dtype)
    f = sj.join_ip if metric == "ip" else sj.join_l2
    a, b = f(Pd, Qd, w.threshold), f(Pd, Qd, w.threshold, recompute=True)
    assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())
    assert sj.count(Pd, Qd, w.threshold, metric) == g.shape[0]


@pytest.mark.parametrize("dtype,d", [("f16", 20), ("f16", 64), ("bf16", 128), ("bf16", 200),
                                     ("i8", 30), ("i8", 64), ("i8", 128), ("i8", 250)])
@pytest.mark.parametrize("metric", ["ip", "l2"])
def test_ordinary_tiles_all_modes(dtype, d, metric):
    """Every resident variant at a size that takes the ordinary tiles (more
    than one for every second CU; smaller joins take the small geometry),
    ragged in both directions, in every mode: the oracle's set, and the same
    array from both second passes of count-then-emit."""
    import paper_2006_12608_amd as sj
    n_p, n_q = 8209, 9001
    w = workloads.random_case(71 + d, n_p, n_q, d, dtype, lo=-3, hi=3, metric=metric)
    rows = np.sort(np.random.default_rng(d).choice(n_p, 500, replace=False))
    x, y = values(dtype, w.P[rows]).astype(np.int64), values(dtype, w.Q).astype(np.int64)
    s = x @ y.T
    if metric == "l2":
        s = (x * x).sum(1)[:, None] + (y * y).sum(1)[None, :] - 2 * s
    w.threshold = float(np.quantile(s, 0.998 if metric == "ip" else 0.002, method="nearest"))
    _, g, _ = run_case(w, rows=rows)
    Pd, Qd = to_device(w.P, dtype), to_device(w.Q, dtype)
    f = sj.join_ip if metric == "ip" else sj.join_l2
    a, b = f(Pd, Qd, w.threshold), f(Pd, Qd, w.threshold, recompute=True)
    assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())
    h = sorted_pairs(a)
    assert np.array_equal(g, h[np.isin(h[:, 0], rows)])
    one = sorted_pairs(f(Pd, Qd, w.threshold, two_pass=False))
    assert np.array_equal(one, h)
    assert sj.count(Pd, Qd, w.threshold, metric) == h.shape[0]


@pytest.mark.parametrize("dtype,d", [("f16", 300), ("bf16", 320), ("f16", 384), ("bf16", 505),
                                     ("i8", 600), ("i8", 640), ("i8", 769)])
@pytest.mark.parametrize("metric", ["ip", "l2"])
@pytest.mark.parametrize("quantile", [0.9995, 0.98, 0.8])
def test_streamed_tiles_all_modes(dtype, d, metric, quantile):
    """The K-streamed kernel at 18 x 19 ragged tiles, more than the CUs, so its
    workgroups go from tile to tile: rows of an odd and an even number of 128-byte
    chunks with and without a partial last one, few and many matches (staged pairs
    that overflow a wave's buffer), in every mode: the oracle's set, and the same
    array from both second passes of count-then-emit."""
    import paper_2006_12608_amd as sj
    n_p, n_q = 4400, 4700
    w = workloads.random_case(81 + d, n_p, n_q, d, dtype, lo=-3, hi=3, metric=metric)
    rows = np.sort(np.random.default_rng(d).choice(n_p, 300, replace=False))
    x, y = values(dtype, w.P[rows]).astype(np.int64), values(dtype, w.Q).astype(np.int64)
    s = x @ y.T
    if metric == "l2":
        s = (x * x).sum(1)[:, None] + (y * y).sum(1)[None, :] - 2 * s
    w.threshold = float(np.quantile(s, quantile if metric == "ip" else 1 - quantile,
                                    method="nearest"))
    _, g, _ = run_case(w, rows=rows)
    Pd, Qd = to_device(w.P, dtype), to_device(w.Q, dtype)
    f = sj.join_ip if metric == "ip" else sj.join_l2
    a, b = f(Pd, Qd, w.threshold), f(Pd, Qd, w.threshold, recompute=True)
    assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())
    h = sorted_pairs(a)
    assert np.array_equal(g, h[np.isin(h[:, 0], rows)])
    one = sorted_pairs(f(Pd, Qd, w.threshold, two_pass=False))
    assert np.array_equal(one, h)
    assert sj.count(Pd, Qd, w.threshold, metric) == h.shape[0]


@pytest.mark.parametrize("dtype,d,metric", [("bf16", 300, "ip"), ("f16", 520, "l2"),
                                             ("i8", 700, "ip"), ("i8", 530, "l2"),
                                             ("bf16", 128, "ip"), ("f16", 256, "l2"),
                                             ("i8", 64, "l2"), ("i8", 40, "ip"),
                                             ("f16", 72, "ip")])
def test_two_pass_match_bits_equal_recompute(dtype, d, metric):
    """Count-then-emit: the second pass that reads the first pass's match bits
    (K-streamed kernel: a bit per result; resident kernel: a record per 32x32
    block with matches) writes the same array (same order) as the one that
    recomputes the product, over several tiles with ragged edges, and the set
    is the oracle's; a capacity one short of the total is an overflow with the
    exact total."""
    import torch
    import paper_2006_12608_amd as sj
    w = workloads.random_case(40 + d, 600, 777, d, dtype, lo=-2, hi=2)
    w.metric = metric
    Pd, Qd = to_device(w.P, dtype), to_device(w.Q, dtype)
    x = values(dtype, w.P).astype(np.int64)
    y = values(dtype, w.Q).astype(np.int64)
    if metric == "ip":
        w.threshold = float(np.quantile(x @ y.T, 0.9, method="nearest"))
    else:
        d2 = (x * x).sum(1)[:, None] + (y * y).sum(1)[None, :] - 2 * (x @ y.T)
        w.threshold = float(np.quantile(d2, 0.1, method="nearest"))
    say("match bits vs recompute", dtype, d, metric, w.threshold)
    ctx = sj.context(0)
    f = sj.join_ip if metric == "ip" else sj.join_l2
    a = f(Pd, Qd, w.threshold, two_pass=True, ctx=ctx)
    st = sj.sj_get_stats(ctx)
    row_bytes = d * (1 if dtype == "i8" else 2)
    assert st.kernel == (2 if row_bytes > 512 else 1) and st.emit_from_bits == 1
    b = f(Pd, Qd, w.threshold, two_pass=True, recompute=True, ctx=ctx)
    assert sj.sj_get_stats(ctx).emit_from_bits == 0
    assert a.shape[0] > 0 and torch.equal(a, b)
    ref = oracle.join(metric, dtype, w.P, w.Q, w.threshold)
    compare(sorted_pairs(a), ref, False)
    c = f(Pd, Qd, w.threshold, two_pass=False, ctx=ctx)
    assert np.array_equal(sorted_pairs(a), sorted_pairs(c))
    total = a.shape[0]
    out = torch.empty((total, 2), dtype=torch.int32, device="cuda")
    with pytest.raises(sj.SjError) as e:
        f(Pd, Qd, w.threshold, cap=total - 1, out=out, two_pass=True, ctx=ctx)
    assert e.value.status == sj.SJ_E_OVERFLOW and e.value.n_out == total


@pytest.mark.parametrize("dtype,d", [("i8", 64), ("bf16", 96)])
@pytest.mark.parametrize("n_p,n_q", [(300, 768), (3500, 10908)])
def test_two_pass_records_every_pair(dtype, d, n_p, n_q):
    """Resident kernel, count-then-emit with every pair matching: every 32x32
    block has a record, and the output is every pair, in the same order as the
    recomputing second pass.  300 x 768 takes the small geometry (a workgroup
    has one tile); at 3500 x 10908 the Q tiles (43 or 86) do not divide by the
    splits of Q, so some workgroups sweep two tiles and fill their records."""
    import torch
    import paper_2006_12608_amd as sj
    w = workloads.random_case(23, n_p, n_q, d, dtype, lo=-3, hi=3)
    Pd, Qd = to_device(w.P, dtype), to_device(w.Q, dtype)
    say("records, every pair", dtype, d, n_p, n_q)
    ctx = sj.context(0)
    a = sj.join_ip(Pd, Qd, -np.inf, two_pass=True, ctx=ctx)
    st = sj.sj_get_stats(ctx)
    assert st.kernel == 1 and st.emit_from_bits == 1
    b = sj.join_ip(Pd, Qd, -np.inf, two_pass=True, recompute=True, ctx=ctx)
    assert torch.equal(a, b)
    del b
    key = a[:, 0].long() * n_q + a[:, 1].long()
    assert torch.equal(key.sort().values, torch.arange(n_p * n_q, device="cuda"))


def test_ties_are_inclusive():
    """Rows with known exact scores at the threshold are reported; one above is not."""
    rng = np.random.default_rng(5)
    for dtype in ("f16", "bf16", "i8"):
        x = rng.integers(-5, 6, size=(40, 24))
        w = workloads.Workload("ties", "ip", dtype, workloads.encode(x, dtype),
                               workloads.encode(x, dtype), 0.0, np.zeros((0, 2), np.int64))
        S = x @ x.T
        for s in (float(S[3, 7]), float(S[3, 7]) + 1):
            run_case(w, thr=s)


def test_empty_and_zero_dim():
    import torch
    import paper_2006_12608_amd as sj
    say("empty inputs")
    P = torch.zeros((0, 16), dtype=torch.float16, device="cuda")
    Q = torch.ones((5, 16), dtype=torch.float16, device="cuda")
    assert sj.join_ip(P, Q, 0.0).shape[0] == 0
    assert sj.join_l2(Q, P, 0.0).shape[0] == 0
    assert sj.count(P, Q, -1.0) == 0
    # d = 0: every score is 0, so everything matches s <= 0 and nothing s > 0
    P0 = torch.zeros((7, 0), dtype=torch.int8, device="cuda")
    Q0 = torch.zeros((9, 0), dtype=torch.int8, device="cuda")
    assert sj.join_ip(P0, Q0, 0.0).shape[0] == 63
    assert sj.join_ip(P0, Q0, 0.5).shape[0] == 0
    assert sj.join_l2(P0, Q0, 0.0).shape[0] == 63


def test_self_join_same_pointer_all_variants():
    for dtype, d in (("f16", 64), ("bf16", 300), ("i8", 64), ("i8", 500)):
        w = workloads.random_case(11, 333, 333, d, dtype, lo=-3, hi=3)
        w.Q = w.P
        w.self_join = True
        x = values(dtype, w.P).astype(np.int64)
        w.threshold = float(np.quantile(x @ x.T, 0.98, method="nearest"))
        for two_pass in (False, True):
            _, g, _ = run_case(w, two_pass=two_pass)
            s = set(map(tuple, g.tolist()))
            assert s == {(j, i) for (i, j) in s}


# --------------------------------------------------- full-size workloads

def _sample_rows(n, k, seed):
    rng = np.random.default_rng(seed)
    return np.sort(rng.choice(n, size=k, replace=False))


def _keys_torch(pairs):
    import torch
    return pairs[:, 0].to(torch.int64) * (1 << 32) + pairs[:, 1].to(torch.int64)


# (workload, sampled rows of P for the false-negative check, two-pass,
#  emitted pairs rescored: "all", or the size of a random sample)
FULL = [("ip_bf16_65536x128", 128, False, "all"),
        ("cos_f16_262144x256", 32, False, "all"),
        ("l2_i8_1048576x64", 64, False, "all"),
        ("ip_bf16_clustered_131072x1024", 16, True, 1_000_000)]


@pytest.mark.parametrize("k,n_rows,two_pass,rescore", FULL)
def test_full_size(k, n_rows, two_pass, rescore):
    """The full workload on the GPU in the launch configuration the benchmark
    uses, checked three ways.
    No false positive anywhere: the oracle rescores every emitted pair (on the
    clustered workload, whose 5.2e8 pairs are too many for the oracle's loops,
    a random sample of 10^6 of them) and each one must pass the exact test
    (real-valued inputs: or lie inside the boundary band).
    No false negative: every planted pair is in the output and no decoy is
    (the int8 workload's 1000 pairs at exactly r^2 = 2000 among the planted,
    its 1000 decoys at 2001), and for a random sample of P's rows the
    oracle's matches against all of Q equal the GPU's.
    No duplicates, and the output size equals sj_count's total."""
    import torch
    import paper_2006_12608_amd as sj
    w = workloads.make_config(k)
    Pd, Qd = to_device(w.P, w.dtype), to_device(w.Q, w.dtype)
    say("full size", w.name, "two_pass", two_pass, "rescore", rescore)
    total = sj.count(Pd, Qd, w.threshold, w.metric)
    out = torch.empty((total, 2), dtype=torch.int32, device="cuda")
    f = sj.join_ip if w.metric == "ip" else sj.join_l2
    pairs = f(Pd, Qd, w.threshold, cap=total, out=out, two_pass=two_pass)
    assert pairs.shape[0] == total
    band = 1e-3 * abs(w.threshold) if w.real_valued else 0.0
    kd = _keys_torch(pairs)
    if rescore == "all":
        gk = np.sort(kd.cpu().numpy().astype(np.uint64))
        assert np.unique(gk).size == gk.size, "duplicate pairs in the GPU output"
        sel = np.stack([(gk >> np.uint64(32)).astype(np.int64),
                        (gk & np.uint64(0xFFFFFFFF)).astype(np.int64)], 1)
    else:
        assert torch.unique(kd).numel() == total, "duplicate pairs in the GPU output"
        rng = np.random.default_rng(91)
        idx = torch.from_numpy(rng.choice(total, size=min(rescore, total), replace=False)).cuda()
        sel = pairs[idx].cpu().numpy().view(np.uint32).astype(np.int64)
        gk = None
    del kd
    sc = oracle.scores(w.metric, w.dtype, w.P, w.Q, sel)
    ok = sc >= w.threshold - band if w.metric == "ip" else sc <= w.threshold + band
    in_band = int(np.sum(np.abs(sc - w.threshold) <= band)) if band else 0
    say("rescored", sel.shape[0], "pairs; failing", int((~ok).sum()), "in band", in_band)
    assert ok.all(), f"false positives: {sel[~ok][:5].tolist()} scores {sc[~ok][:5].tolist()}"
    if w.planted.size:
        pk = keys(w.planted)
        assert np.isin(pk, gk).all(), "planted pairs missing"
    if w.decoys.size:
        assert not np.isin(keys(w.decoys), gk).any(), "decoys reported"
        ties = oracle.scores(w.metric, w.dtype, w.P, w.Q, w.planted[-(w.decoys.shape[0]):])
        assert np.all(ties == w.threshold)   # the exact ties are among the planted pairs
    rows = _sample_rows(w.n_p, n_rows, 77 + workloads.NAMES.index(k))
    if w.planted.size:   # include some planted rows
        rows = np.unique(np.concatenate([rows, w.planted[:4, 0]]))
    sel_rows = torch.isin(pairs[:, 0], torch.from_numpy(rows.astype(np.int32)).cuda())
    g = sorted_pairs(pairs[sel_rows])
    ref = oracle.join(w.metric, w.dtype, w.P, w.Q, w.threshold, rows=rows, band=band)
    info = compare(g, ref, w.real_valued)
    say("total", total, "rows", rows.size, "sampled matches", ref.total, info)
