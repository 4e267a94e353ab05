"""Fields whose outlier, word and run counts together are 2^32 or nearly: compressed
and read back within the bound (up to 17 GB of input and about 95 GB on the device)."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,codec", [(4_294_000_000, "huffman"), (4_294_000_000, "auto"), (4_289_728_809, "huffman"),
                                     (4_294_960_000, "huffman")])
def test_one_column(n, codec):
    from paper_2105_12912_amd import ebc as E

    eb = 1e-2
    if torch.cuda.mem_get_info()[0] < 100e9:
        pytest.skip("needs 100 GB of free device memory")
    g = torch.Generator(device="cuda").manual_seed(7)
    block = torch.randn(1 << 20, generator=g, device="cuda").cumsum(0) / 300
    if codec == "auto":  # long runs
        block[:-70000] = 0.0
    x = torch.zeros(n, device="cuda")
    for a in range(0, n, block.numel()):
        x[a:a + block.numel()] = block[:n - a] * (1 if (a >> 20) % 3 else -1)
    p = E.make_params(eb, "abs", codec=codec)
    out = torch.empty(6 << 30, dtype=torch.uint8, device="cuda")
    ws = torch.empty(E.ebc_compress_workspace_size(2, (1, n), p), dtype=torch.uint8, device="cuda")
    st, size = E.ebc_compress(x.data_ptr(), 2, (1, n), p, out.data_ptr(), out.numel(), ws.data_ptr(), ws.numel(),
                              E._stream_handle())
    assert st == 0 and size > 0
    del ws
    torch.cuda.empty_cache()
    print("compressed", size, flush=True)
    a = out[:size]
    assert E.ebc_archive_info(E.archive_header(a))["codec"] == (0 if codec == "huffman" else 1)
    y = E.decompress(a, workspace=E.Workspace("cuda")).reshape(-1)
    for k in range(0, n, 1 << 28):
        assert float((y[k:k + (1 << 28)] - x[k:k + (1 << 28)]).abs().max()) <= eb
    del x, y, out
    torch.cuda.empty_cache()


@pytest.mark.parametrize("n", [2_300_000_000, 4_294_900_000])
def test_runs_of_one(n):
    """Run indices above 2^31 in the searches of decompression, for the tiles and for
    the codes of outliers."""
    from paper_2105_12912_amd import ebc as E

    eb = 0.4
    if torch.cuda.mem_get_info()[0] < 150e9:
        pytest.skip("needs 150 GB of free device memory")
    x = torch.zeros(n, device="cuda")
    x[1::2] = 1.0
    x[n - 100] = x[n // 3] = x[7] = 2000.0
    p = E.make_params(eb, "abs", codec="rle")
    out = torch.empty(E.HDR_BYTES + 6 * n + 4096, dtype=torch.uint8, device="cuda")
    ws = torch.empty(E.ebc_compress_workspace_size(1, (n,), p), dtype=torch.uint8, device="cuda")
    st, size = E.ebc_compress(x.data_ptr(), 1, (n,), p, out.data_ptr(), out.numel(), ws.data_ptr(), ws.numel(),
                              E._stream_handle())
    assert st == 0 and size > 6 * n - 4096
    del ws
    torch.cuda.empty_cache()
    print("compressed", size, flush=True)
    y = E.decompress(out[:size], workspace=E.Workspace("cuda"))
    for k in range(0, n, 1 << 28):
        assert float((y[k:k + (1 << 28)] - x[k:k + (1 << 28)]).abs().max()) <= eb
    del x, y, out
    torch.cuda.empty_cache()
