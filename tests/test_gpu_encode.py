"""The Huffman write pass against the oracle over codeword lengths: pairs, fours
and eights of neighbours that fit 32 and 64 bits and that do not, for every
chunk size that gives a lane another number of symbols."""
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


def codes(kind, n, rng):
    if kind == "short":    # about 1 bit each
        return np.where(rng.random(n) < 0.01, rng.integers(1, 1024, n), 512)
    if kind == "flat":     # 10 bits each: eights of 80 bits
        return rng.integers(1, 1024, n)
    # lengths from 1 to above 20, long ones next to each other in places
    c = 512 + np.minimum(rng.geometric(0.5, n), 24)
    for a in rng.integers(0, max(1, n - 16), max(1, n // 5000)):
        c[a:a + 12] = 600 + np.arange(12)[: n - a]
    return c


@pytest.mark.parametrize("hc", [64, 128, 256, 512, 1024, 2048, 8192])
@pytest.mark.parametrize("kind", ["short", "flat", "long"])
@pytest.mark.parametrize("n", [5, 1023, 100_001, 2_000_000])
def test_codeword_lengths(E, n, kind, hc):
    d = codes(kind, n, np.random.default_rng(n)).astype(np.int64) - 512
    x = np.zeros(n)
    full = n // 256 * 256
    x[:full] = np.cumsum(d[:full].reshape(-1, 256), axis=1).reshape(-1)
    x[full:] = np.cumsum(d[full:])
    x *= 0.02
    want = O.compress(x, 0.01, "abs", codec="huffman", hc=hc)
    a = E.compress(torch.from_numpy(x).cuda(), 0.01, "abs", codec="huffman", huff_chunk=hc)
    assert a.cpu().numpy().tobytes() == want


@pytest.mark.parametrize("hc,together", [(64, 64), (64, 61), (256, 64)])
def test_chunk_of_longest_codewords(E, hc, together):
    """Frequencies like Fibonacci's on top of 64 symbols that occur once give these
    33 bits each: side by side they are a chunk of more than 32 bits per symbol."""
    below, total, counts = 64, 64 + 65, [65]
    while len(counts) < 27:  # each just above the total of all but the last
        counts.append(below + 2)
        below, total = total, total + counts[-1]
    small = [(k + 1) // 2 * (1 - 2 * (k % 2)) for k in range(27)]  # the most frequent: 0
    d = np.repeat(np.array(small[::-1], dtype=np.int8), counts)
    np.random.default_rng(1).shuffle(d)
    rare = np.stack([np.arange(14, 46), -np.arange(14, 46)], axis=1).reshape(-1).astype(np.int8)
    at = 128 * 1024
    d = np.concatenate([d[:at], rare[:together], d[at:], rare[together:]])
    n = d.size
    x = np.zeros(n, dtype=np.float32)
    full = n // 256 * 256
    x[:full] = (np.cumsum(d[:full].reshape(-1, 256), axis=1, dtype=np.int32) * 0.02).reshape(-1)
    x[full:] = np.cumsum(d[full:], dtype=np.int32) * 0.02
    want = O.compress(x, 0.01, "abs", codec="huffman", hc=hc)
    lens = np.frombuffer(want, np.uint8, 1024, 128)
    assert lens.max() == 33 and (lens == 33).sum() == 64
    a = E.compress(torch.from_numpy(x).cuda(), 0.01, "abs", codec="huffman", huff_chunk=hc)
    assert a.cpu().numpy().tobytes() == want
    y = E.decompress(a).cpu().numpy()
    assert np.abs(y.astype(np.float64) - x).max() <= 0.01
