"""The Huffman decoder against the oracle where its paths part: sub-chunk and
chunk sizes, streams of one workgroup size or another, last groups that are
not full, codewords longer than the first and the second table level."""
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


def walk(n, kind, seed):
    """Steps whose quantised sizes give short, mixed or very skewed code lengths."""
    rng = np.random.default_rng(seed)
    if kind == "flat":  # codewords of equal length
        s = rng.integers(-400, 401, n)
    elif kind == "long":  # a geometric tail: codewords of 1 to above 20 bits
        s = np.minimum(rng.geometric(0.5, n), 200) * rng.choice([-1, 1], n)
    else:  # mostly zeros
        s = (rng.random(n) < 0.02) * rng.integers(-300, 301, n)
    x = np.zeros(n)
    for a in range(0, n, 256):  # a chunk predicts from zero
        x[a:a + 256] = np.cumsum(s[a:a + 256])
    return (x * 0.02).astype(np.float32)


def check(E, x, hc, n_bins=1024):
    want = O.compress(x, 0.01, "abs", codec="huffman", hc=hc, n_bins=n_bins)
    a = E.compress(torch.from_numpy(x).cuda(), 0.01, "abs", codec="huffman", huff_chunk=hc, n_bins=n_bins)
    assert a.cpu().numpy().tobytes() == want
    y = E.decompress(a).cpu().numpy()
    assert y.tobytes() == O.decompress(want).tobytes()


@pytest.mark.parametrize("kind", ["flat", "long", "zeros"])
@pytest.mark.parametrize("hc", [64, 256, 1024, 65536])
@pytest.mark.parametrize("n", [1, 33, 257, 64 * 256, 64 * 256 + 1, 70_001])
def test_small_streams(E, n, hc, kind):
    check(E, walk(n, kind, n + hc), hc)


@pytest.mark.parametrize("kind", ["flat", "long", "zeros"])
@pytest.mark.parametrize("groups", [768, 769, 2049, 4097])
def test_workgroup_sizes(E, groups, kind):
    # 64-symbol chunks: a group is 4096 symbols
    check(E, walk(groups * 4096 - 77, kind, groups), 64)


def test_many_bins(E):
    check(E, walk(300_003, "flat", 3), 1024, n_bins=65536)


@pytest.mark.parametrize("kind", ["flat", "long"])
@pytest.mark.parametrize("subs", [31, 32, 33, 127, 129, 65_536, 65_537])
def test_half_waves(E, subs, kind):
    # up to 65536 sub-chunks, 32 to a wave and 128 to a workgroup; sub-chunks of 64
    check(E, walk(subs * 64 - 5, kind, subs), 64)
