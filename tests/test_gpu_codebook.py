"""Codebook and decoder tables against the oracle over histograms that pick
their paths: few and many used symbols (one or several sorted batches per wave,
LDS and scratch sorts), equal counts, counts of one to four digits, geometric
and Fibonacci-like tails (long codewords, merge rounds with a single pair) and
merge rounds with more than 64 leaves or nodes."""
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


def codes_field(codes, n_bins):
    """A 1D field whose quant-codes are the given ones (chunks of 256)."""
    d = codes.astype(np.int64) - n_bins // 2
    x = np.zeros(d.size)
    for a in range(0, d.size, 256):
        x[a:a + 256] = np.cumsum(d[a:a + 256])
    return x.astype(np.float64) * 0.02


def symbols(kind, used, n_bins, rng):
    s = rng.permutation(np.arange(1, n_bins))[:used]
    if kind == "equal":
        f = np.full(used, 7)
    elif kind == "ones":
        f = np.ones(used, int)
        f[0] = 70_000
    elif kind == "geometric":
        f = np.maximum(1, (200_000 * 0.7 ** np.arange(used))).astype(int)
    elif kind == "fibonacci":
        f = np.ones(used, int)
        for k in range(2, min(used, 24)):
            f[k] = f[k - 1] + f[k - 2]
    else:
        f = rng.integers(1, 60, used)
    c = np.repeat(s, f)
    return rng.permutation(c)


@pytest.mark.parametrize("kind", ["equal", "ones", "geometric", "fibonacci", "random"])
@pytest.mark.parametrize("n_bins,used", [(1024, 1), (1024, 2), (1024, 3), (1024, 64), (1024, 65), (1024, 130),
                                         (1024, 1023), (4096, 1025), (4096, 4095), (8192, 300), (8192, 5000),
                                         (32768, 16384), (32768, 16385), (65536, 30000)])
def test_codebook(E, n_bins, used, kind):
    rng = np.random.default_rng(n_bins + used)
    c = symbols(kind, used, n_bins, rng)
    x = codes_field(c, n_bins)
    want = O.compress(x, 0.01, "abs", codec="huffman", n_bins=n_bins)
    a = E.compress(torch.from_numpy(x).cuda(), 0.01, "abs", codec="huffman", n_bins=n_bins)
    assert a.cpu().numpy().tobytes() == want
    y = E.decompress(a).cpu().numpy()
    assert y.tobytes() == O.decompress(want).tobytes()
