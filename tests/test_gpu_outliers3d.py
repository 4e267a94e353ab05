"""3D reconstruction around outliers, against the oracle: every row alignment,
block edge and outlier density that picks another path of the kernels
(chunks without outliers, flagged chunks, partial chunks along each axis)."""
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


def field(shape, density, dtype):
    """A smooth field; `density` of its elements are pushed far away."""
    x = synth.grf_field(shape, 5).astype(dtype)
    rng = np.random.default_rng(7)
    x[rng.random(shape) < density] += dtype(40.0)
    x.flat[0], x.flat[-1] = -50.0, 50.0  # outliers in the first and the last chunk
    return x


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("density", [0.0, 0.002, 0.3])
@pytest.mark.parametrize("shape", [(8, 8, 256), (16, 32, 512), (9, 33, 261), (7, 8, 260), (17, 9, 515),
                                   (8, 41, 7), (24, 16, 64)])
def test_outliers_by_alignment_and_density(E, shape, density, dtype):
    x = field(shape, density, dtype)
    want = O.compress(x, 0.01, "abs", n_bins=64)
    a = E.compress(torch.from_numpy(x).cuda(), 0.01, "abs", n_bins=64)
    assert a.cpu().numpy().tobytes() == want
    y = E.decompress(a).cpu().numpy()
    assert y.tobytes() == O.decompress(want).tobytes()


def test_codes_of_every_value_are_told_from_outliers(E):
    """65536 bins: codes from 1 to 65535, the centre 32768 among them."""
    shape = (16, 16, 256)
    rng = np.random.default_rng(3)
    q = rng.integers(1, 65536, size=shape).astype(np.uint16)
    q[:, :8, :128] = 32768
    qd = torch.from_numpy(q.view(np.int16).reshape(-1)).cuda()
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    got = E.debug_reconstruct(qd, none, none, 3, shape[::-1], 65536, 1.0).cpu().numpy()
    d = (q.astype(np.int64) - 32768).reshape(2, 8, 2, 8, 32, 8)
    for ax in (1, 3, 5):
        d = d.cumsum(axis=ax)
    assert np.array_equal(got.reshape(shape), d.reshape(shape).astype(np.float32))


@pytest.mark.parametrize("shape", [(8, 8, 256), (9, 10, 11)])
def test_outlier_code_without_a_listed_outlier_is_refused(E, shape):
    n = int(np.prod(shape))
    q = np.full(n, 32, np.int16)
    q[n // 2] = 0
    none = torch.empty(0, dtype=torch.int32, device="cuda")
    with pytest.raises(E.EbcError) as ei:
        E.debug_reconstruct(torch.from_numpy(q).cuda(), none, none, 3, shape[::-1], 64, 1.0)
    assert ei.value.status == E.EBC_ERR_ARCHIVE


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("density", [0.0, 0.05])
@pytest.mark.parametrize("shape", [(1, 16, 512), (1, 9, 261), (2, 8, 66), (3, 7, 63), (9, 1, 4), (5, 3, 1), (1, 1, 70)])
def test_few_planes_rows_and_columns(E, shape, density, dtype):
    """A last plane without its pair, blocks of one row, quads that the field cuts."""
    x = field((16, 16, 512), density, dtype)[tuple(slice(0, n) for n in shape)].copy()
    x.flat[0], x.flat[-1] = -50.0, 50.0
    want = O.compress(x, 0.01, "abs", n_bins=64)
    a = E.compress(torch.from_numpy(x).cuda(), 0.01, "abs", n_bins=64)
    assert a.cpu().numpy().tobytes() == want
    y = E.decompress(a).cpu().numpy()
    assert y.tobytes() == O.decompress(want).tobytes()
