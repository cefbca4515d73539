"""The layers with costs held in registers (schedule 1, up to 4096 distinct values):
every F_i[j] bit for bit the minimum over all predecessors (sampled columns against the
oracle, every column against the layer-by-layer schedule), at the edges of the 1024
predecessors of a thread's slot and of the column counts per workgroup, and the
codebook that the traceback finds."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import pipeline
from paper_2608_18147_amd import ecasq, inputs

pytestmark = pytest.mark.gpu


def _distinct(x, n):
    _, at = np.unique(x.astype(np.float32), return_index=True)
    return x.astype(np.float32)[np.sort(at)][:n]


CASES = [(257, 3), (264, 40), (1000, 16), (1024, 5), (1025, 64), (1032, 8), (2048, 33), (2049, 12),
         (3071, 64), (3072, 9), (3073, 12),
         (4095, 6), (4096, 64)]


@pytest.mark.parametrize("p,s", CASES)
@pytest.mark.parametrize("kind", ["normal", "integers", "outlier"])
def test_held_layers(p, s, kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if kind == "integers":  # many equal candidates: the lowest predecessor counts
        x = np.arange(p, dtype=np.float32)
    else:
        x = _distinct(inputs.normal(p + 400, 9), p)
        if kind == "outlier":
            x[0], x[1] = 1e30, -1e6
    H = pipeline.prepare(x)
    assert H.p == p
    xd = torch.from_numpy(np.ascontiguousarray(x)).to("cuda")
    rng = np.random.default_rng(p)
    z = np.zeros(p)
    for lam in (0.0, 0.01, 1.0):
        print("[case] held", kind, p, s, lam, flush=True)
        F, K, _, _, res = ecasq.ecasq_dp_trace(xd, s, lam, schedule=1)
        F, K = F.cpu().numpy(), K.cpu().numpy()
        for i in range(2, s + 1):
            cols = np.unique(np.concatenate([rng.integers(i - 1, p, 16),
                                             [i - 1, i, p - 1, p - 8, p - 9, 1023, 1024]]))
            cols = cols[(cols >= i - 1) & (cols < p)]
            lamp = lam * H.s2tot
            Fo = (pipeline.dp_columns(H, 2, lamp, cols=cols) if i == 2 else
                  pipeline.dp_columns(H, i, lamp, F[i - 1], z, z, cols))[0]
            np.testing.assert_array_equal(F[i, cols], Fo, err_msg=f"{p} {lam} layer {i}")
            assert np.all(np.isinf(F[i, : i - 1])) or i == 2
        # every column against the layer-by-layer schedule
        F0, K0, _, _, res0 = ecasq.ecasq_dp_trace(xd, s, lam, schedule=0)
        F0, K0 = F0.cpu().numpy(), K0.cpu().numpy()
        for i in range(2, s + 1):
            np.testing.assert_array_equal(F[i, i - 1:p], F0[i, i - 1:p], err_msg=f"layer {i}")
            np.testing.assert_array_equal(K[i, i - 1:p], K0[i, i - 1:p], err_msg=f"layer {i}")
        assert res[:4] == res0[:4]
        # the codebook along the argmins of every layer
        cb, rk, info = ecasq.ecasq_solve_lagrangian(
            xd, s, lam, options=ecasq.ecasq_default_options(refine_rounds=0))
        t = res[3]
        chain = [p - 1]
        for i in range(int(t), 2, -1):
            chain.append(int(K[i, chain[-1]]))
        np.testing.assert_array_equal(rk.cpu().numpy(), ([0] + chain[::-1]))
