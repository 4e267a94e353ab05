"""Compression into buffers that are too small, by one byte or by nearly all: refused
with the size that is needed, nothing stored past the end, the fields beside it whole."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("codec", ["huffman", "rle", "rle_vle"])
@pytest.mark.parametrize("short", [1, 5000, None])
def test_refused(short, codec):
    from paper_2105_12912_amd import ebc as E
    from paper_2105_12912_amd.batch import BatchCompress

    x = np.random.default_rng(3).standard_normal((300, 1700)).astype(np.float32)
    want = O.compress(x, 1e-4, n_bins=64, codec=codec)
    cap = len(want) - short if short else 128
    b = BatchCompress([torch.from_numpy(x).cuda() for _ in range(5)], 1e-4, n_bins=64, codec=codec)
    for i in (0, 2, 4):
        b.descs[i].out_cap = cap
    for _ in range(3):
        for o in b.outs:
            o.fill_(0xA5)
        b.launch()
        for i, (size, status, _) in enumerate(b.results()):
            if i % 2:
                assert status == 0 and b.outs[i][:size].cpu().numpy().tobytes() == want
            else:
                assert status == E.EBC_ERR_OUT_TOO_SMALL and size == 0
                assert bool((b.outs[i][cap:] == 0xA5).all())
    rank, dims = E.field_rank_dims(b.fields[0])
    ws = E.Workspace("cuda")
    st, size = E.ebc_compress(b.fields[0].data_ptr(), rank, dims, b.params, b.outs[0].data_ptr(), cap,
                              *ws.get(E.ebc_compress_workspace_size(rank, dims, b.params)), E._stream_handle())
    assert st == E.EBC_ERR_OUT_TOO_SMALL and size == 0 and f"({len(want)} bytes needed)" in E.ebc_last_error()
