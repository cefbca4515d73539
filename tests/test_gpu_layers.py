"""The layers with bounds (schedule 1 above 4096 distinct values and 64 per
layer): every F_i[j] must be the minimum over all predecessors bit for bit, so
no bound may discard one that holds it.  Sampled columns of every layer against
the oracle's recomputation, which scans every predecessor of the GPU's previous
layer; sizes at the edges of the 16- and 64-column workgroups and on both sides
of the size where one takes the other's place, and values that make the bounds
loose or the prefix sums cancel."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

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
    ("normal_4112", lambda: _distinct(inputs.normal(5000, 2), 4112), 33),
    ("lognormal_6145", lambda: _distinct(inputs.lognormal_signed(7000, 3), 6145), 64),
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
    assert p > 4096 and p > 64 * s, "sizes that take the layers with bounds"
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
