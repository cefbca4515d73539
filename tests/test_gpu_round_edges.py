"""Rounding (ecasq_quantize) at the edges of its kernels: parts of the four
entries of a thread, both sides of the size that one workgroup takes, inputs that
are not aligned, every storage type, and the 32-bit search and comparison
where they are closest to the 64-bit ones: codebook values between floats, beyond
the floats' range, repeated, a float apart and at zero's two signs."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import pipeline
from paper_2608_18147_amd import ecasq

pytestmark = pytest.mark.gpu


def _check(xd, q, seed):
    x = xd.float().cpu().numpy()
    sym, ent, hist = ecasq.ecasq_quantize(xd, torch.from_numpy(q), seed)
    s_o, h_o, e_o = pipeline.quantize(x, q, seed)
    np.testing.assert_array_equal(sym.cpu().numpy(), s_o)
    np.testing.assert_array_equal(hist.cpu().numpy(), h_o)
    # 256 terms of h, each within a few ulp
    assert abs(float(ent) - e_o) <= 1e-12 * max(1.0, abs(e_o))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 4097, 32767, 32768, 32769, 40962,
                               (1 << 22) - 1, (1 << 22) + 3])
def test_round_sizes(d, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] round", d, dtype, flush=True)
    g = np.random.default_rng(d)
    x = torch.from_numpy(g.standard_normal(d + 1).astype(np.float32)).to("cuda").to(dtype)[1:]
    for t in (1, 2, 3, 9, 255, 256) if d < 10 ** 6 else (16, 256):
        q = np.sort(g.standard_normal(t)) * 2.0
        _check(x, q, 2 ** 35 + d)


BOOKS = {
    "between_floats": np.array([-1.0 - 1e-9, -1e-9, 1e-9, 1.0 + 1e-9, 1.0 + 2e-9]),
    "a_float_apart": np.array([1.0, 1.0 + 2.0 ** -23, 1.0 + 2.0 ** -22, 2.0]),
    "zeros_and_denormals": np.array([-1e-45, -0.0, 0.0, 1e-60, 1.4e-45, 1.0]),
    "beyond_floats": np.array([-1e300, -1e39, 0.0, 1e39, 1e300]),
    "narrow_interval": np.array([0.0, 1e-40, 2.0]),
    "repeated": np.array([-1.0, 0.5, 0.5, 0.5, 1.0]),
}


@pytest.mark.parametrize("name", sorted(BOOKS))
def test_round_books(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] book", name, flush=True)
    q = BOOKS[name]
    g = np.random.default_rng(1)
    f = q.astype(np.float32)[np.abs(q) < 1e38]
    near = np.concatenate([f, np.nextafter(f, np.float32(9)), np.nextafter(f, np.float32(-9)),
                           np.float32([0.0, -0.0, 1e-45, -1e-45, 3e38, -3e38])])
    x = np.concatenate([np.tile(near, 40), g.standard_normal(2000).astype(np.float32),
                        (1.0 + g.random(2000) * 2.0 ** -21).astype(np.float32)])
    for n in (x.size, 40000):
        _check(torch.from_numpy(np.resize(x, n)).to("cuda"), q, 77)
