"""3D reconstruction of a last layer of one to four planes, whose waves take two or
four blocks along x: block edges along x, layers below it, every row alignment."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2105_12912_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("density", [0.0, 0.1])
@pytest.mark.parametrize("yx", [(9, 64), (8, 65), (17, 130), (3, 193), (16, 256), (7, 261), (1, 515)])
@pytest.mark.parametrize("nz", [1, 2, 3, 4, 5, 9, 10, 11, 12, 20])
def test_last_layer(nz, yx, density, dtype):
    from paper_2105_12912_amd import ebc as E

    x = synth.grf_field((32, 32, 1024), 5)[:nz, :yx[0], :yx[1]].astype(dtype)
    rng = np.random.default_rng(nz)
    x[rng.random(x.shape) < density] += dtype(40.0)
    x.flat[0], x.flat[-1] = -50.0, 50.0  # outliers in the first and the last chunk
    want = O.compress(x, 0.01, "abs", n_bins=64)
    a = E.compress(torch.from_numpy(x).cuda(), 0.01, "abs", n_bins=64)
    assert a.cpu().numpy().tobytes() == want
    y = E.decompress(a).cpu().numpy()
    assert y.tobytes() == O.decompress(want).tobytes()
