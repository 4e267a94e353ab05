"""Round trips and error reports of one-field decompression on the current and
on another stream: the same field, and the same error text, as with statistics."""
import pytest
import torch

from paper_2105_12912_amd import ebc

pytestmark = pytest.mark.gpu


def report(*args, **kw):
    with pytest.raises(ebc.EbcError) as e:
        ebc.decompress(*args, **kw)
    assert e.value.status == ebc.EBC_ERR_ARCHIVE
    return str(e.value)


@pytest.mark.parametrize("side", [False, True])
def test_status(side):
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(70001, generator=g, device="cuda").cumsum(0)
    a = ebc.compress(x, 1e-3, codec="huffman").clone()
    torch.cuda.synchronize()
    stream = torch.cuda.Stream() if side else None
    ref, st = ebc.decompress(a, stats=True)
    assert torch.equal(ebc.decompress(a, stream=stream), ref) and st.out_bytes == a.numel()
    short = a[:-16].clone()             # refused by the host
    wrong = a.clone()                   # refused on the device: bit count of the first sub-chunk
    wrong[128 + 1024:128 + 1026] = 255
    torch.cuda.synchronize()
    for bad in (short, wrong):
        assert report(bad, stream=stream) == report(bad, stats=True)
    assert torch.equal(ebc.decompress(a, stream=stream), ref)
