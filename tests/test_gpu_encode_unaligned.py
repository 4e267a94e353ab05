"""Archives written to a buffer that starts at any byte: the same bytes, also where a
chunk takes more than 32 bits per symbol."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2105_12912_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def compress_at(x, offset, eb, mode, **kw):
    from paper_2105_12912_amd import ebc as E

    p = E.make_params(eb, mode, dtype=E._dtype_code(x), **kw)
    buf = torch.zeros(E.ebc_compress_bound(*E.field_rank_dims(x), p) + 16, dtype=torch.uint8, device="cuda")
    a = E.compress(x, eb, mode, out=buf[offset:], **kw)
    assert a.data_ptr() == buf.data_ptr() + offset
    return a.cpu().numpy().tobytes()


@pytest.mark.parametrize("offset", [1, 2, 4, 7])
@pytest.mark.parametrize("codec", ["huffman", "rle", "rle_vle"])
def test_any_byte(codec, offset):
    x = synth.lognormal_3d((24, 40, 33), 5)
    assert compress_at(torch.from_numpy(x).cuda(), offset, 1e-3, "rel", codec=codec) == O.compress(x, 1e-3, codec=codec)


def longest_codewords(hc):
    """Frequencies like Fibonacci's on top of hc symbols that occur once, which fill
    one chunk and take more than 32 bits each."""
    below, total, counts = hc, 2 * hc + 1, [hc + 1]
    while len(counts) < 34 - hc.bit_length():  # each just above the total of all but the last
        counts.append(below + 2)
        below, total = total, total + counts[-1]
    small = [(k + 1) // 2 * (1 - 2 * (k % 2)) for k in range(len(counts))]  # the most frequent: 0
    d = np.repeat(np.array(small[::-1], dtype=np.int16), counts)
    np.random.default_rng(1).shuffle(d)
    k = np.arange(hc // 2, dtype=np.int16) + 17
    at = 128 * 1024
    d = np.concatenate([d[:at], np.stack([k, -k], axis=1).reshape(-1), d[at:]])
    x = np.zeros(d.size, dtype=np.float32)
    full = d.size // 256 * 256
    x[:full] = (np.cumsum(d[:full].reshape(-1, 256), axis=1, dtype=np.int32) * 0.02).reshape(-1)
    x[full:] = np.cumsum(d[full:], dtype=np.int32) * 0.02
    return x


@pytest.mark.parametrize("hc,offset", [(64, 1), (64, 6), (512, 3)])
def test_chunk_above_32_bits_per_symbol(hc, offset):
    x = longest_codewords(hc)
    want = O.compress(x, 0.01, "abs", codec="huffman", hc=hc)
    y = O.huffman_layout(x.size, 1024, hc, 0)
    bits = np.frombuffer(want, np.uint16, y["n_sub"], y["sbits"]).astype(np.int64)
    at, hs = 128 * 1024 // min(hc, 256), hc // min(hc, 256)
    assert bits[at:at + hs].sum() > 32 * hc  # the chunk of the rare ones
    assert compress_at(torch.from_numpy(x).cuda(), offset, 0.01, "abs", codec="huffman", huff_chunk=hc) == want
