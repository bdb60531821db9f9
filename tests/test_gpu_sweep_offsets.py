"""The sweep's key-row offsets at the largest slices (``-m gpu``): 32-bit ones up to 4 GiB of rows, 64-bit beyond."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Wk", [8191, 8192], ids=["last_slice_under_4GiB", "slice_of_4GiB"])
@pytest.mark.parametrize("sep", [0, 2], ids=["plain", "second_run"])
def test_scores_belong_to_the_map(scram, Wk, sep):
    """Every score the sweeps return is the dot product with the row their map names, on a slice whose last
    rows lie just below, or reach, 4 GiB; the best of many draws lies in each half of the slice for some query."""
    Hq, Wq, Hk, d = 16, 24, 4096, 64
    gen = torch.Generator(device="cuda").manual_seed(7)
    K = torch.empty(1, Hk, Wk, d, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    Q = torch.randn(1, Hq, Wq, d, device="cuda", generator=gen).to(torch.bfloat16)
    first = scram.patchmatch(Q, K, 2, 5)
    prev = first[None].contiguous() if sep else None
    J, s = scram.patchmatch(Q, K, 3, 5, return_score=True, prev=prev, sep=max(sep, 1))
    rows = K.reshape(Hk * Wk, d)[J.reshape(-1).long()].double()
    want = (rows * Q.reshape(-1, d).double()).sum(1)
    mag = (rows * Q.reshape(-1, d).double()).abs().sum(1)
    assert ((s.reshape(-1).double() - want).abs() <= 40 * 2.0 ** -24 * mag).all()  # 40 roundings of sum |q k|
    assert (J < Hk * Wk // 2).any() and (J >= Hk * Wk // 2).any()
