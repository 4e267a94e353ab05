"""Batched compression where the counts of some fields are never written (a constant
field, one with a NaN, the words of a run-length coded one): the offsets of the
fields behind them start anywhere modulo 2^32 and wrap inside a field's stream."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2105_12912_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def uncoded(kind):
    x = np.zeros(20_000, dtype=np.float32)
    if kind == "nan":
        x[77] = np.nan
    elif kind == "runs":
        x[5_000:] = 1.0
    return x


@pytest.mark.parametrize("fill", [0xFF, 0xFE, 0x00])
@pytest.mark.parametrize("codec", ["auto", "auto_vle"])
@pytest.mark.parametrize("kind", ["const", "nan", "runs"])
def test_offsets_behind_uncoded_fields(kind, codec, fill):
    from paper_2105_12912_amd.batch import BatchCompress

    fields = [uncoded(kind), synth.random_walk_1d(50_001, 3), uncoded(kind), synth.smooth_2d(130, 96, 4),
              synth.lognormal_3d((24, 40, 33), 5)]
    b = BatchCompress([torch.from_numpy(x).cuda() for x in fields], 1e-3, codec=codec)
    b.ws.fill_(fill)  # 0xFF: each count that is not written counts as -1
    b.launch()
    for i, (x, (size, status, _)) in enumerate(zip(fields, b.results())):
        if kind == "nan" and i in (0, 2):
            assert status == -6 and size == 0
            continue
        assert status == 0
        assert b.outs[i][:size].cpu().numpy().tobytes() == O.compress(x, 1e-3, codec=codec), f"field {i}"
