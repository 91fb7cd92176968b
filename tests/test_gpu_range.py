"""pmc_range against numpy: sizes around its workgroups' shares, samples that
are not finite, rows that are not 16-byte aligned, and a workspace of the
smallest size the call takes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHARE = 4 * 1024  # samples one workgroup takes at least


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [1, 3, 255, SHARE - 1, SHARE + 1, 256 * SHARE - 1, 256 * SHARE + 5, 2_500_001])
@pytest.mark.parametrize("skip", [0, 1])
def test_range_matches_numpy(n, dtype, skip):
    import torch

    from paper_2308_11759_amd import pmc

    rng = np.random.Generator(np.random.PCG64(n + skip))
    x = rng.normal(0.0, 1.0, size=n + skip).astype(dtype)
    special = rng.integers(0, n + skip, size=min(5, n // 2))
    x[special] = np.array([np.nan, np.inf, -np.inf, -0.0, np.finfo(dtype).max], dtype=dtype)[:len(special)]
    xd = torch.from_numpy(x).to("cuda:0")[skip:]
    x = x[skip:]
    fin = x[np.isfinite(x)].astype(np.float64)
    want = (fin.min(), fin.max(), int((~np.isfinite(x)).sum()))
    assert pmc.Context(0).range(xd) == want


def test_range_nothing_finite():
    import torch

    from paper_2308_11759_amd import pmc

    lo, hi, bad = pmc.Context(0).range(torch.full((70, 60), float("nan"), device="cuda:0"))
    assert np.isnan(lo) and np.isnan(hi) and bad == 4200
