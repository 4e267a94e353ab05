"""2D reconstruction against the oracle: tile widths and row alignments, fields
narrower than a chunk, rows and columns past the last whole chunk, outliers from
none to all, single precision and double."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2105_12912_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def E():
    from paper_2105_12912_amd import ebc
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ebc.lib()
    return ebc


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("density", [0.0, 0.002, 0.4, 1.0])
@pytest.mark.parametrize("shape", [(1, 1), (1, 300), (300, 1), (16, 16), (17, 15), (33, 64), (40, 65), (31, 131), (16, 256),
                                   (50, 260), (129, 515)])
def test_shapes_and_densities(E, shape, density, dtype):
    x = (synth.grf_field(shape, 9) if min(shape) > 1 else np.zeros(shape)).astype(dtype)
    rng = np.random.default_rng(5)
    pick = rng.random(shape) < density
    x[pick] += (rng.standard_normal(shape) * 100)[pick].astype(dtype)
    want = O.compress(x, 0.01, "abs", n_bins=64)
    a = E.compress(torch.from_numpy(x).cuda(), 0.01, "abs", n_bins=64)
    assert a.cpu().numpy().tobytes() == want
    assert E.decompress(a).cpu().numpy().tobytes() == O.decompress(want).tobytes()
