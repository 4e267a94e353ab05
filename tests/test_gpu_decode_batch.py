"""A batched decompression on either side of as many 1024-lane decode workgroups as
the device holds at once (one per CU), each field by itself as the expectation."""
import pytest

torch = pytest.importorskip("torch")
from paper_2105_12912_amd import ebc
from paper_2105_12912_amd.batch import BatchCompress, BatchDecompress

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extra", [-1, 0, 1, 40])
def test_workgroups_around_the_cus(extra):
    k = torch.cuda.get_device_properties(0).multi_processor_count + extra
    g = torch.Generator(device="cuda")
    g.manual_seed(extra + 2)
    # above 2048 groups of 64 sub-chunks in all, fields of one workgroup each
    steps = torch.randn(k, 140_000, generator=g, device="cuda")
    fields = [x[: 139_000 + 7 * i % 900].cumsum(0).contiguous() for i, x in enumerate(steps)]
    c = BatchCompress(fields, 1e-4)
    c.launch()
    arcs = c.archives()
    d = BatchDecompress(arcs)
    for o in d.outs:
        o.fill_(float("nan"))
    d.launch()
    assert d.statuses() == [0] * k
    for x, a, o in zip(fields, arcs, d.outs):
        assert torch.equal(ebc.decompress(a).view(torch.int32), o.view(torch.int32))
        x = x.double()
        assert (o.double() - x).abs().max() <= 1e-4 * (x.max() - x.min())
