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
