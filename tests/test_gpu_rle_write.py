"""Run-length encoding against the oracle where its write pass parts: runs over
many tiles, tiles without a run start, a start at every element, ends in the
same thread, wave, tile or a later one; fields whose workspace holds the
run-start flags and fields that read the codes again; long Huffman chunks (the
passes then get launches of their own)."""
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


def field(n, kind):
    """fp32 values whose quant-codes (chunks of 256) are mostly one value."""
    rng = np.random.default_rng(n)
    d = np.zeros(n)
    if kind == "changes":
        d = rng.integers(-1, 2, n).astype(float)
    elif kind == "rare":
        k = max(1, n // 5000)
        d[rng.integers(0, n, k)] = 1.0
    elif kind == "last":
        d[-1] = 1.0
    x = np.zeros(n)
    for a in range(0, n, 256):
        x[a:a + 256] = np.cumsum(d[a:a + 256])
    x[0] += 3.0  # a value range, also for "one"
    return (x * 0.02).astype(np.float32)


def check(E, x, **opt):
    want = O.compress(x, 0.01, "abs", codec=opt["codec"], n_bins=opt.get("n_bins", 1024),
                      hc=opt.get("huff_chunk", 1024))
    a = E.compress(torch.from_numpy(x).cuda(), 0.01, "abs", **opt)
    assert a.cpu().numpy().tobytes() == want
    assert E.decompress(a).cpu().numpy().tobytes() == O.decompress(want).tobytes()


@pytest.mark.parametrize("codec", ["rle", "rle_vle"])
@pytest.mark.parametrize("n_bins,hc", [(1024, 1024), (16, 1024), (1024, 4096)])
@pytest.mark.parametrize("kind", ["one", "changes", "rare", "last"])
@pytest.mark.parametrize("n", [1, 16, 17, 1024, 4096, 4097, 100_003])
def test_runs(E, n, kind, n_bins, hc, codec):
    check(E, field(n, kind), codec=codec, n_bins=n_bins, huff_chunk=hc)


@pytest.mark.parametrize("n_bins", [16, 1024])
def test_flags_on_a_large_field(E, n_bins):
    check(E, field((1 << 24) + 4099, "rare"), codec="rle", n_bins=n_bins)


@pytest.mark.parametrize("codec", ["rle", "rle_vle"])
@pytest.mark.parametrize("runs", [1022, 1024, 1026, 4096])
@pytest.mark.parametrize("n", [8191, 8192, 30_001])
def test_runs_of_one_tile(E, n, runs, codec):
    """Tiles of few runs around one of as many as given, which picks who writes them."""
    d = np.zeros(n)
    d[4096:min(n, 4096 + runs):2] = 1.0
    d[0] = 3.0
    x = np.zeros(n)
    for a in range(0, n, 256):
        x[a:a + 256] = np.cumsum(d[a:a + 256])
    check(E, (x * 0.02).astype(np.float32), codec=codec)
