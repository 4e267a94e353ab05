"""The outlier list of a compression against the oracle, over segment lengths
(tile widths), row alignments and densities, partial segments at row ends."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def E():
    from paper_2105_12912_amd import ebc
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ebc.lib()
    return ebc


@pytest.mark.parametrize("density", [0.001, 0.2, 1.0])
@pytest.mark.parametrize("shape", [(1,), (255,), (70001,), (33, 7), (40, 65), (19, 523), (300, 128), (9, 10, 31),
                                   (17, 9, 100), (8, 16, 261)])
def test_outlier_list(E, shape, density):
    rng = np.random.default_rng(11)
    x = rng.standard_normal(shape).astype(np.float32)
    x[rng.random(shape) < density] *= np.float32(1e4)
    want = O.compress(x, 0.5, "abs", n_bins=64)
    got = E.compress(torch.from_numpy(x).cuda(), 0.5, "abs", n_bins=64).cpu().numpy().tobytes()
    assert got == want


@pytest.mark.parametrize("shape", [(900, 2), (900, 8), (700, 9), (300, 16), (300, 17), (9, 40, 1), (9, 40, 8), (10, 33, 15)])
def test_short_rows(E, shape):
    """Rows shorter than a segment, one to four lanes each."""
    rng = np.random.default_rng(12)
    x = rng.standard_normal(shape).astype(np.float32)
    x[rng.random(shape) < 0.4] *= np.float32(1e4)
    want = O.compress(x, 0.5, "abs", n_bins=64)
    got = E.compress(torch.from_numpy(x).cuda(), 0.5, "abs", n_bins=64).cpu().numpy().tobytes()
    assert got == want
