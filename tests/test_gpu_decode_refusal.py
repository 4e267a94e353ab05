"""Corrupt Huffman streams that only the decoder itself can tell: refused, whichever
workgroup meets the fault first, and without harm to the other fields of a batch."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_faults_in_many_workgroups():
    """Twelve fields whose decode workgroups are more than the device holds at once
    (those of a field that start late see the fault that early ones found)."""
    from paper_2105_12912_amd import ebc as E
    from paper_2105_12912_amd.batch import BatchDecompress

    n, bins = 4_000_000, 64
    g = torch.Generator(device="cuda").manual_seed(2)
    x = torch.randn(n, generator=g, device="cuda").cumsum(0)
    good = E.compress(x, 1e-3, n_bins=bins, codec="huffman", huff_chunk=64).clone()
    want = E.decompress(good)
    host = good.cpu().numpy()
    at = O.huffman_layout(n, bins, 64, 0)["sbits"]
    arcs = []
    for i in range(12):
        a = host.copy()
        if i % 3:  # bit counts one too small, in every chunk or in a few
            bits = a[at:at + 2 * (n // 64)].view(np.uint16)
            pick = (np.arange(bits.size) % (1 if i % 3 == 1 else 5001) == 0) & (bits % 32 != 1)
            bits[pick] -= 1
        arcs.append(torch.from_numpy(a).cuda())
    d = BatchDecompress(arcs)
    for _ in range(3):
        d.launch()
        assert d.statuses() == [0 if i % 3 == 0 else E.EBC_ERR_ARCHIVE for i in range(12)]
        for i in range(0, 12, 3):
            assert torch.equal(d.outs[i], want)


def wrapped(n, bins, chunk_words):
    """A Huffman archive of n symbols in chunks of 64 whose stored bit counts make
    chunk_words words each; the header holds their sum modulo 2^32, and as many words
    follow."""
    h = O.huffman_layout(n, bins, 64, 0)
    words = (n // 64 * chunk_words) % (1 << 32)
    size = h["words"] + (4 * words + 15) // 16 * 16
    a = np.zeros(size, np.uint8)
    a[:O.HDR_BYTES] = np.frombuffer(O.compress(np.arange(1000, dtype=np.float32), 0.1, "abs", n_bins=bins,
                                               codec="huffman", hc=64), np.uint8)[:O.HDR_BYTES]
    a[16:40] = np.array([n, 1, 1], np.uint64).view(np.uint8)
    a[88:120] = np.array([0, n // 64, words, size], np.uint64).view(np.uint8)
    a[h["len"]:h["len"] + 2] = 1
    a[h["sbits"]:h["sbits"] + 2 * (n // 64)] = np.full(n // 64, min(32 * chunk_words, 65535), np.uint16).view(np.uint8)
    return a


@pytest.mark.parametrize("n,chunk_words", [(1 << 27, 2048), (1 << 28, 1024), ((1 << 27) + 64 * 1000, 2048)])
def test_word_counts_that_wrap(n, chunk_words):
    from paper_2105_12912_amd import ebc as E

    a = wrapped(n, 16, chunk_words)
    assert O.decompress_status(a.tobytes()) == E.EBC_ERR_ARCHIVE
    assert E.decompress_status(torch.from_numpy(a).cuda()) == E.EBC_ERR_ARCHIVE
