"""1D run-length coded fields, reconstructed from their runs: tile and chunk
edges, tiles inside one run, of a few and of more runs than are staged, outliers,
both value types, outputs that are not 16-byte aligned, and several in one batch."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def field(n, kind, dtype, seed=0):
    rng = np.random.default_rng(n + seed)
    d = np.zeros(n)
    if kind == "steps":     # a few runs per tile, some outliers
        at = rng.integers(0, n, max(1, n // 700))
        d[at] = rng.integers(-900, 901, at.size)
    elif kind == "dense":   # a run per one or two elements
        d = rng.integers(-3, 4, n).astype(float)
    x = np.cumsum(d) % 4000 * 0.02
    x[-1] += 0.02           # never constant
    return x.astype(dtype)


@pytest.mark.parametrize("codec", ["rle", "rle_vle"])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind", ["one", "steps", "dense"])
@pytest.mark.parametrize("n", [2, 255, 257, 1023, 4096, 4097, 70_003])
def test_round_trip(n, kind, dtype, codec):
    from paper_2105_12912_amd import ebc as E
    x = field(n, kind, dtype)
    want = O.compress(x, 0.01, "abs", codec=codec)
    a = E.compress(torch.from_numpy(x).cuda(), 0.01, "abs", codec=codec)
    assert a.cpu().numpy().tobytes() == want
    ref = O.decompress(want).tobytes()
    assert E.decompress(a).cpu().numpy().tobytes() == ref
    # an output one element off the 16-byte grid; its neighbours stay
    buf = torch.full((n + 2,), 7.0, dtype=E.decompress(a).dtype, device="cuda")
    E.decompress(a, out=buf[1:n + 1])
    got = buf.cpu().numpy()
    assert got[1:-1].tobytes() == ref and got[0] == 7 and got[-1] == 7


def test_batch():
    from paper_2105_12912_amd import ebc as E
    from paper_2105_12912_amd.batch import BatchDecompress
    xs = [field(n, k, dt, i) for i, (n, k, dt) in enumerate(
        [(9001, "steps", np.float32), (4096, "one", np.float64), (20_000, "dense", np.float32)])]
    xs.insert(1, field(10_000, "steps", np.float32, 9).reshape(100, 100))
    arcs = [E.compress(torch.from_numpy(x).cuda(), 0.01, "abs", codec=c).clone()
            for x, c in zip(xs, ["rle", "rle", "rle_vle", "huffman"])]
    d = BatchDecompress(arcs)
    d.capture()
    for _ in range(3):
        for o in d.outs:
            o.zero_()
        d.replay()
        torch.cuda.synchronize()
        for o, a in zip(d.outs, arcs):
            assert o.cpu().numpy().tobytes() == O.decompress(a.cpu().numpy().tobytes()).tobytes()
