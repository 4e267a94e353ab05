"""Construction of fields whose rows are shorter than a quad, beside the shortest that
hold one, with few and with many outliers."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n_bins", [64, 8192])
@pytest.mark.parametrize("density", [0.01, 0.6])
@pytest.mark.parametrize("rows", [(1001,), (17, 133), (9, 8)])
@pytest.mark.parametrize("nx", [1, 2, 3, 4, 5])
def test_narrow_rows(nx, rows, density, n_bins, dtype):
    from paper_2105_12912_amd import ebc as E

    rng = np.random.default_rng(nx)
    x = rng.standard_normal(rows + (nx,)) * 0.1
    x[rng.random(x.shape) < density] += 0.08 * n_bins
    x = x.astype(dtype)
    want = O.compress(x, 0.05, "abs", n_bins=n_bins)
    a = E.compress(torch.from_numpy(x).cuda(), 0.05, "abs", n_bins=n_bins)
    assert a.cpu().numpy().tobytes() == want
    assert E.decompress(a).cpu().numpy().tobytes() == O.decompress(want).tobytes()
