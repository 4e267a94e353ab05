"""Value range of fp64 fields on both sides of the size up to which the range
pass keeps the field in the last-level cache: extremes and non-finite values
anywhere, the tail unit included."""
import pytest

torch = pytest.importorskip("torch")
from paper_2105_12912_amd import ebc

pytestmark = pytest.mark.gpu

KEEP = 20_000_000


@pytest.mark.parametrize("n", [16384, 16385, KEEP, KEEP + 1, KEEP + 3 * 16384])
def test_range(n):
    x = torch.zeros(n, dtype=torch.float64, device="cuda")
    places = [0, 1, 4097, 16383, n // 2, n - 16385, n - 2, n - 1]
    for k, (i, j) in enumerate(zip(places, places[1:] + places[:1])):
        if min(i, j) < 0 or i == j:
            continue
        x[i], x[j] = -1.5 - k, 2.25 + k
        _, st = ebc.compress(x, 1e-2, stats=True)
        assert (st.value_min, st.value_max) == (-1.5 - k, 2.25 + k)
        x[i] = x[j] = 0.0


@pytest.mark.parametrize("n", [16385, KEEP, KEEP + 1])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
def test_nonfinite(n, bad):
    x = torch.zeros(n, dtype=torch.float64, device="cuda")
    x[n // 3] = 1.0
    for i in (0, 16383, n - 1):
        x[i] = bad
        with pytest.raises(ebc.EbcError) as e:
            ebc.compress(x, 1e-2)
        assert e.value.status == ebc.EBC_ERR_NONFINITE
        x[i] = 0.0
