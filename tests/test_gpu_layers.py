"""The layers with bounds (schedule 1 above 4096 distinct values, few layers to
them): every F_i[j] must be the minimum over all predecessors bit for bit, so
no bound may discard one that holds it.  Sampled columns of every layer against
the oracle's recomputation, which scans every predecessor of the GPU's previous
layer; sizes at the edges of the 16- and 64-column workgroups and on both sides
of the size where one takes the other's place, and values that make the bounds
loose or the prefix sums cancel."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from bench import schedule_kernel
from oracle import pipeline
from paper_2608_18147_amd import ecasq, inputs

pytestmark = pytest.mark.gpu


def _distinct(x, n):
    """The first n distinct values of x, in x's order."""
    _, at = np.unique(x.astype(np.float32), return_index=True)
    return x.astype(np.float32)[np.sort(at)][:n]


def _clusters(n):
    """Runs of adjacent floats between wide gaps: steep counts per width."""
    rng = np.random.default_rng(3)
    base = rng.standard_normal(n // 50 + 1).astype(np.float32)
    x = np.repeat(base, 50)[:n].view(np.int32) + np.tile(np.arange(50), n // 50 + 1)[:n]
    return x.astype(np.int32).view(np.float32)


def _wide(n):
    rng = np.random.default_rng(4)
    return (rng.standard_normal(n) * 10.0 ** rng.integers(-30, 30, n)).astype(np.float32)


def _outliers(n, big):
    x = inputs.normal(n, 5)
    x[0], x[1] = big, -big
    return x


CASES = [
    ("normal_4097", lambda: _distinct(inputs.normal(5000, 1), 4097), 20),
    ("normal_4112", lambda: _distinct(inputs.normal(5000, 2), 4112), 21),
    ("lognormal_6145", lambda: _distinct(inputs.lognormal_signed(7000, 3), 6145), 47),
    ("integers_5000", lambda: np.arange(5000, dtype=np.float32), 24),
    ("clusters_6000", lambda: _distinct(_clusters(6400), 6000), 16),
    ("wide_range_6000", lambda: _distinct(_wide(6200), 6000), 12),
    ("outlier_1e6_5000", lambda: _outliers(5000, 1e6), 12),
    ("outlier_1e30_5000", lambda: _outliers(5000, 1e30), 12),
    ("student_t_49151", lambda: _distinct(inputs.student_t(50500, 6), 49151), 12),
    ("student_t_49152", lambda: _distinct(inputs.student_t(50500, 6), 49152), 12),
    ("weights_49217", lambda: _distinct(inputs.weight_mixture(51000, 7), 49217), 40),
    ("clusters_50000", lambda: _distinct(_clusters(51200), 50000), 12),
    ("outlier_1e30_50000", lambda: _outliers(50000, 1e30), 6),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_layers_hold_every_minimum(case):
    name, make, s = case
    x = make()
    H = pipeline.prepare(x)
    p = H.p
    assert schedule_kernel(p, s)[0] == "k_layer"
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    xd = torch.from_numpy(np.ascontiguousarray(x)).to("cuda")
    rng = np.random.default_rng(11)
    z = np.zeros(x.size)
    for lam in (0.0, 0.003, 0.2, 50.0):
        print("[case]", name, "p", p, "s", s, "lambda", lam, flush=True)
        F = ecasq.ecasq_dp_trace(xd, s, lam, schedule=1, argmins=False)[0].cpu().numpy()
        for i in range(2, s + 1):
            n = 24 if p < 10000 else 10
            cols = np.unique(np.concatenate([
                rng.integers(i - 1, p, n), [i - 1, i, p - 1, p - 2, p - 17, p - 65]]))
            cols = cols[(cols >= i - 1) & (cols < p)]
            lamp = lam * H.s2tot
            if i == 2:
                Fo = pipeline.dp_columns(H, 2, lamp, cols=cols)[0]
            else:
                Fo = pipeline.dp_columns(H, i, lamp, F[i - 1], z, z, cols)[0]
            np.testing.assert_array_equal(F[i, cols], Fo, err_msg=f"{name} {lam} layer {i}")
            if i < 4:  # columns no chain of i values reaches
                assert np.all(np.isinf(F[i, : i - 1])) or i == 2


def _cancelled(n, centre, spread, big):
    """Values around centre and one entry that takes their prefix sums with it."""
    x = (centre + spread * np.random.default_rng(13).standard_normal(n)).astype(np.float32)
    x[7] = big
    return x


@pytest.mark.parametrize("big", [-1e16, -1e18, 1e20, -1e20, -1e30])
@pytest.mark.parametrize("centre,spread", [(1.0, 0.1), (10.0, 1.0), (1000.0, 1.0)])
@pytest.mark.parametrize("n,s", [(6000, 8), (53000, 5)])
def test_layers_where_sums_cancel(n, s, centre, spread, big):
    """Sums rounded to 53 bits leave frequencies far outside [0, 1] here, and entropy terms
    far below 0: every column of every layer against the layer-by-layer schedule, which
    evaluates every predecessor, and the codebooks of the two."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = _cancelled(n, centre, spread, big)
    xd = torch.from_numpy(x).to("cuda")
    p = np.unique(x).size
    assert schedule_kernel(p, s)[0] == "k_layer"
    opts = [ecasq.ecasq_default_options(dp_schedule=1, refine_rounds=0),
            ecasq.ecasq_default_options(dp_schedule=0, recovery=1, refine_rounds=0)]
    for lam in (0.0, 0.003, 0.2, 50.0):
        print("[case] cancelled", n, s, centre, spread, big, lam, flush=True)
        F1, _, _, _, r1 = ecasq.ecasq_dp_trace(xd, s, lam, schedule=1, argmins=False)
        F0, _, _, _, r0 = ecasq.ecasq_dp_trace(xd, s, lam, schedule=0)
        for i in range(2, s + 1):
            bad = int((F1[i, i - 1:p] != F0[i, i - 1:p]).sum())
            assert bad == 0, f"lambda {lam} layer {i}: {bad} columns"
        assert r1[0] == r0[0] and r1[3] == r0[3]
        (c1, k1, i1), (c0, k0, i0) = (ecasq.ecasq_solve_lagrangian(xd, s, lam, options=o)
                                      for o in opts)
        assert torch.equal(k1, k0) and torch.equal(c1, c0) and i1["mse"] == i0["mse"]


@pytest.mark.parametrize("kind", ["narrow", "narrow_rare", "offset", "outlier"])
@pytest.mark.parametrize("m,s", [(5000, 6), (8000, 9)])
def test_layers_on_a_uniform_grid(m, s, kind):
    """A grid's points are 53-bit values: on a narrow range far from zero its steps lie far
    below an ulp of the entries.  The codebooks of the two schedules."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(m)
    n = 20000
    if kind == "narrow":
        x = 1.0 + 2.0 ** -23 * rng.integers(0, 3, n)
    elif kind == "narrow_rare":
        x = np.full(n, 1.0 + 2.0 ** -23)
        x[:5] = 1.0
    elif kind == "offset":
        x = 1000.0 + rng.standard_normal(n)
    else:
        x = 5.0 + rng.standard_normal(n)
        x[3] = -1e20
    xd = torch.from_numpy(x.astype(np.float32)).to("cuda")
    for lam in (0.0, 0.01, 1.0):
        print("[case] grid", kind, m, s, lam, flush=True)
        (c1, k1, i1), (c0, k0, i0) = (
            ecasq.ecasq_solve_lagrangian(xd, s, lam, options=ecasq.ecasq_default_options(
                alphabet=1, alphabet_size=m, refine_rounds=0, **kw))
            for kw in (dict(dp_schedule=1), dict(dp_schedule=0, recovery=1)))
        assert schedule_kernel(i1["p"], s)[0] == "k_layer"
        assert torch.equal(k1, k0) and torch.equal(c1, c0) and i1["mse"] == i0["mse"]


@pytest.mark.parametrize("n,s", [(20000, 16), (70000, 24)])
def test_layers_that_give_up(n, s):
    """Values over 60 decades leave the bounds nothing to hold: the layers stop and the solve
    comes again by the sweep.  Each entry point's result against the layer-by-layer
    schedule, with the next solve enqueued ahead (below 2^16 values) and without."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = _wide(n)
    assert schedule_kernel(np.unique(x).size, s)[0] == "k_layer"
    xd = torch.from_numpy(x).to("cuda")

    def opt(**kw):
        return ecasq.ecasq_default_options(max_search_passes=4, **kw)

    def same(a, b):
        assert torch.equal(a[1], b[1]) and torch.equal(a[0], b[0])
        for k in ("t", "lambda", "mse", "entropy", "entropy_surrogate", "dp_solves", "status"):
            assert a[2][k] == b[2][k], k

    top = ecasq.ecasq_solve_lagrangian(xd, s, 0.0, options=opt(refine_rounds=0))
    b = 0.6 * top[2]["entropy_surrogate"]
    ecasq.ecasq_timing_enable(True)
    try:
        print("[case] give up, budget", n, s, b, flush=True)
        ecasq.ecasq_timing_read(ecasq.TIMING_SWEEP, reset=True)
        got = ecasq.ecasq_solve(xd, s, b, options=opt())
        runs = ecasq.ecasq_timing_read(ecasq.TIMING_SWEEP, reset=True)[1]
        assert got[2]["dp_solves"] > 1 and runs > got[2]["dp_solves"], "a solve has given up"
        same(got, ecasq.ecasq_solve(xd, s, b, options=opt(dp_schedule=0, recovery=1)))
        print("[case] give up, fixed multiplier", n, s, flush=True)
        ecasq.ecasq_timing_read(ecasq.TIMING_SWEEP, reset=True)
        got = ecasq.ecasq_solve_lagrangian(xd, s, 0.01, options=opt())
        assert ecasq.ecasq_timing_read(ecasq.TIMING_SWEEP, reset=True)[1] == 2
        same(got, ecasq.ecasq_solve_lagrangian(xd, s, 0.01,
                                               options=opt(dp_schedule=0, recovery=1)))
    finally:
        ecasq.ecasq_timing_enable(False)
    print("[case] give up, two budgets", n, s, flush=True)
    two = [ecasq.ecasq_solve_budgets(xd, s, [b, 0.8 * b], options=opt(**kw))
           for kw in ({}, dict(dp_schedule=0, recovery=1))]
    for a, b in zip(*two):
        same(a, b)
