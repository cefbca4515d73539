"""Sort, histogram and exact prefix sums (ecasq_histogram) where one launch takes
the general path's place: both sides of 1024 and 4096 entries, every storage type,
values from subnormals to the largest, both zeros and repeats; and entries that are not
finite."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import pipeline
from paper_2608_18147_amd import ecasq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("d", [1, 2, 3, 63, 64, 1023, 1024, 1025, 2049, 4095, 4096, 4097])
def test_prep_sizes(d, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("[case] prep", d, dtype, flush=True)
    g = np.random.default_rng(d)
    wide = 6 if dtype == torch.float16 else 37
    x = g.standard_normal(d) * 10.0 ** g.integers(-wide, min(wide, 4 if wide == 6 else 37), d)
    x[g.integers(0, d, d // 3)] = 0.5
    if d > 8:
        x[:4] = [0.0, -0.0, 1e-45, -1e-45]
    xd = torch.from_numpy(x.astype(np.float32)).to("cuda").to(dtype)
    xd = torch.where(torch.isfinite(xd), xd, torch.ones_like(xd))
    got = [a.cpu().numpy() for a in ecasq.ecasq_histogram(xd)]
    H = pipeline.prepare(xd.float().cpu().numpy())
    assert len(got[0]) == H.p
    for a, b in zip(got, (H.v, H.N, H.S, H.S2)):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("d", [1, 1000, 4096])
@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
def test_prep_reports_nonfinite(d, bad):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = torch.ones(d, device="cuda")
    x[d - 1] = bad
    with pytest.raises(ecasq.EcasqError) as e:
        ecasq.ecasq_histogram(x)
    assert e.value.status == ecasq.ECASQ_ENONFINITE


def test_prep_more_than_1024_tiles():
    """More key tiles than one step of a digit's scan takes (1024): the sorted values
    and counts against torch's sort, the sums within the rounding of a 64-bit sum of
    n terms of one sign, n 2^-53 of it."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    d = (1 << 22) + 4097
    print("[case] prep", d, flush=True)
    x = torch.rand(d, generator=torch.Generator("cuda").manual_seed(5), device="cuda")
    v, N, S, S2 = ecasq.ecasq_histogram(x)
    u, c = torch.unique(x, return_counts=True)
    assert torch.equal(v, u.double())
    assert torch.equal(N, torch.cumsum(c, 0).double())
    t = torch.cumsum(u.double() * c, 0)
    assert bool(((S - t).abs() <= d * 2.0 ** -53 * t + 1e-300).all())
