"""The fp32 key side of the backward on the matrix cores, against the oracle (``-m gpu``)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import tile_maps, to_dev

pytestmark = pytest.mark.gpu

# square 8 x 8 key tiles with ragged edges, 64 x 1 and 4 x 16 ones, the smallest grids, two grids
GRIDS = [(2, 21, 13, 21, 13), (1, 70, 1, 70, 1), (2, 5, 70, 3, 67), (1, 3, 5, 3, 5), (1, 9, 31, 30, 22)]
# 128 channels, 64 with several maps and 17 x 17 windows take the lane-group kernels: controls
WIDTHS = [(16, 3), (16, 9), (32, 5), (64, 3), (64, 15), (64, 17), (128, 3), (128, 7)]


@pytest.mark.parametrize("d,window", WIDTHS)
@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
def test_f32_key_strips(scram, d, window, grid):
    S, Hq, Wq, Hk, Wk = grid
    rng = np.random.default_rng(d + 7 * window + Hq)
    Q, dO = (rng.standard_normal((S, Hq, Wq, d)).astype(np.float32) for _ in range(2))
    K, V = (rng.standard_normal((S, Hk, Wk, d)).astype(np.float32) for _ in range(2))
    dev = [to_dev(x, "f32") for x in (Q, K, V)]
    m = tile_maps(S, Hq, Wq, Hk, Wk, rng)
    # one map; entries of one key beyond a chunk (constant); two and three maps, repeated and distant
    sets = [m[n][None] for n in ("random", "coherent", "constant", "two_far")]
    sets += [np.stack([m["coherent"], m["outliers"]]), np.stack([m["coherent"], m["coherent"], m["random"]])]
    for J in sets:
        for causal in ((False, True) if (Hq, Wq) == (Hk, Wk) else (False,)):
            got = scram.sparse_attend_backward(*dev, torch.from_numpy(J).cuda(), to_dev(dO, "f32"), window, causal=causal)
            ref = oracle.sparse_attend_backward(Q, K, V, J, window, d ** -0.5, dO, flags=oracle.CAUSAL if causal else 0)
            for name, g, r in zip(("dQ", "dK", "dV"), got, ref):
                err = np.abs(g.double().cpu().numpy() - r).max() / max(np.abs(r).max(), 1e-30)
                assert err <= 2e-5, (name, J.shape[0], causal, err)  # the bar of the other backward tests


@pytest.mark.parametrize("d", [16, 64])
def test_non_finite_gradients_stay_with_their_keys(scram, d):
    """A query whose output gradient holds an infinity or a NaN reaches exactly the keys of its windows,
    although the key side reads entries in chunks that the keys of a strip share."""
    S, H, W, window = 1, 24, 24, 3
    rng = np.random.default_rng(d)
    Q, K, V, dO = (to_dev(rng.standard_normal((S, H, W, d)).astype(np.float32), "f32") for _ in range(4))
    J = torch.arange(H * W, dtype=torch.int32, device="cuda").reshape(S, H, W)
    clean = scram.sparse_attend_backward(Q, K, V, J, dO, window)
    dO[0, 5, 6, 3] = float("inf")
    dO[0, 17, 20, 1] = float("nan")
    got = scram.sparse_attend_backward(Q, K, V, J, dO, window)
    near = torch.zeros(S, H, W, dtype=torch.bool, device="cuda")
    for u, v in ((5, 6), (17, 20)):
        near[0, u - 1:u + 2, v - 1:v + 2] = True
    for g, c in zip(got[1:], clean[1:]):
        assert torch.isfinite(g[~near]).all()
        # the same sums in either order of the entries
        assert torch.allclose(g[~near], c[~near], rtol=1e-5, atol=2e-5 * float(c.abs().max()))
        assert (~torch.isfinite(g[near])).any(dim=-1).all()


def key_sets(J, H, W, window, causal):
    """[queries, keys] of one slice: whether the union of the query's windows holds the key."""
    b, n = window // 2, H * W
    k = np.arange(n)
    held = np.zeros((n, n), bool)
    for m in J.reshape(len(J), n):
        held |= (np.abs(m[:, None] // W - k[None] // W) <= b) & (np.abs(m[:, None] % W - k[None] % W) <= b)
    return held & (k[None] <= k[:, None]) if causal else held


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,kappa,window", [(16, 1, 5), (16, 3, 3), (32, 2, 5), (32, 3, 7), (64, 1, 7)])
def test_non_finite_gradients_of_unions(scram, d, kappa, window, causal):
    """The same with several maps, the causal mask and keys that gather hundreds of entries (more than the 128
    that are summed in one run): the keys of the affected queries' sets, and no others."""
    H, W = 24, 24
    rng = np.random.default_rng(d + kappa)
    Q, K, V, dO = (rng.standard_normal((1, H, W, d)).astype(np.float32) for _ in range(4))
    own = np.arange(H * W).reshape(1, H, W)
    # the queries' own keys, then three quarters of the queries at one key (an early one, so that the mask keeps it)
    many = np.where(rng.random((1, H, W)) < 0.75, 2 * W + 3, rng.integers(0, H * W, (1, H, W)))
    J = np.stack([many, own, np.roll(own, 5, 2)][:kappa]).astype(np.int32)
    ref = oracle.sparse_attend_backward(Q, K, V, J, window, d ** -0.5, dO, flags=oracle.CAUSAL if causal else 0)
    bad = {17 * W + 20: (3, np.inf), 9 * W + 6: (d - 1, np.nan)}
    for q, (ch, x) in bad.items():
        dO[0, q // W, q % W, ch] = x
    got = scram.sparse_attend_backward(*(to_dev(x, "f32") for x in (Q, K, V)), torch.from_numpy(J).cuda(),
                                       to_dev(dO, "f32"), window, causal=causal)
    held = key_sets(J, H, W, window, causal)
    assert max(held.sum(0)) > 3 * 128
    near = held[list(bad)].any(0)
    assert near.any() and not near.all()
    for name, g, r in zip(("dK", "dV"), got[1:], ref[1:]):
        g, r = g.double().cpu().numpy().reshape(H * W, d), r.reshape(H * W, d)
        assert np.isfinite(g[~near]).all(), name
        assert np.abs(g[~near] - r[~near]).max() <= 2e-5 * np.abs(r).max(), name
        assert (~np.isfinite(g[near])).any(1).all(), name
    # dV of a key in a set is not finite in that channel, and only there
    dv = got[2].cpu().numpy().reshape(H * W, d)
    for q, (ch, _) in bad.items():
        assert not np.isfinite(dv[held[q], ch]).any()
    rest = np.ones(d, bool)
    rest[[ch for ch, _ in bad.values()]] = False
    assert np.isfinite(dv[:, rest]).all()


@pytest.mark.parametrize("grid", [(24, 24), (5, 70), (90, 1), (1, 90)], ids=lambda g: "x".join(map(str, g)))
@pytest.mark.parametrize("d,kappa,window", [(16, 1, 3), (16, 3, 5), (32, 2, 3), (64, 1, 5), (64, 2, 3), (128, 1, 3)])
def test_sets_of_one_key_leave_dK_alone(scram, d, kappa, window, grid):
    """Where the causal mask leaves a query one key, its weight is 1 and dS is 0: the key's dK is exactly 0 and its dV
    the query's dO, if no other query holds it."""
    H, W = grid
    S, b, rng = 8, window // 2, np.random.default_rng(d + kappa + H)
    Q, K, V, dO = (to_dev(4 * rng.standard_normal((S, H, W, d)), "f32") for _ in range(4))
    i = np.arange(H * W)
    # windows that reach back to the query's own key and no further; the second map repeats it, the third holds no key
    # that the mask keeps, except for the last queries
    after = np.minimum(i // W + (b if H > 1 else 0), H - 1) * W + np.minimum(i % W + (b if W > 1 else 0), W - 1)
    J = np.stack([after, after, np.full(H * W, H * W - 1)][:kappa]).astype(np.int32)
    held = key_sets(J, H, W, window, True)
    lone = held.sum(1) == 1
    keys = np.flatnonzero((held[lone].sum(0) == 1) & (held[~lone].sum(0) == 0))
    assert len(keys) > H * W // 8
    owner = held[:, keys].argmax(0)
    Jd = torch.from_numpy(np.broadcast_to(J.reshape(kappa, 1, H, W), (kappa, S, H, W)).copy()).cuda()
    dQ, dK, dV = (x.cpu().reshape(S, H * W, d) for x in
                  scram.sparse_attend_backward(Q, K, V, Jd, dO, window, causal=True))
    assert not dK[:, keys].any()
    assert torch.equal(dV[:, keys], dO.cpu().reshape(S, H * W, d)[:, owner])
    assert not dQ[:, np.flatnonzero(lone)].any()


@pytest.mark.parametrize("d,kappa,window", [(16, 1, 3), (16, 2, 5), (32, 1, 7), (32, 3, 3), (64, 1, 3), (64, 1, 15)])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("many", [128, 129, 1025, 2200])
def test_strips_that_a_team_sums(scram, d, kappa, window, causal, many):
    """Keys that many queries share, by one wave up to 128 entries of a strip and by 8 waves above: one entry more,
    more than eight chunks for each of the waves, a remainder."""
    H = W = 48
    rng = np.random.default_rng(many + d)
    Q, K, V, dO = (rng.standard_normal((1, H, W, d)).astype(np.float32) for _ in range(4))
    q = np.arange(H * W)
    # the other queries at the grid's end
    J = np.stack([np.where(q < many, (5 + 9 * c) * W + 6, H * W - 1 - q % 200) for c in range(kappa)])
    J = J.reshape(kappa, 1, H, W).astype(np.int32)
    dev = [to_dev(x, "f32") for x in (Q, K, V)]
    got = scram.sparse_attend_backward(*dev, torch.from_numpy(J).cuda(), to_dev(dO, "f32"), window, causal=causal)
    ref = oracle.sparse_attend_backward(Q, K, V, J, window, d ** -0.5, dO, flags=oracle.CAUSAL if causal else 0)
    for name, g, r in zip(("dQ", "dK", "dV"), got, ref):
        err = np.abs(g.double().cpu().numpy() - r).max() / np.abs(r).max()
        assert err <= 2e-5, (name, err)  # the bar of the other backward tests


def _us(fn, n=10):
    for _ in range(3):
        fn()
    best = float("inf")
    for _ in range(5):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(n):
            fn()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / n * 1e3)
    return best


def test_time_of_shared_keys_and_of_rows_that_are_not_finite(scram):
    """A map that takes all queries to one key, and one NaN in dO, against the queries' own keys and finite rows.
    Measured: 18 and 1.7 times the time; 80 and 10 where one wave sums all entries of a strip and where the keys of a
    strip that is not finite are summed one by one."""
    H, d = 128, 64
    gen = torch.Generator(device="cuda").manual_seed(5)
    Q, K, V, dO = (torch.randn(1, H, H, d, device="cuda", generator=gen) for _ in range(4))
    own = torch.arange(H * H, dtype=torch.int32, device="cuda").reshape(1, H, H)
    one = torch.full_like(own, H * H // 2 + H // 2)
    base = _us(lambda: scram.sparse_attend_backward(Q, K, V, own, dO, 3))
    assert _us(lambda: scram.sparse_attend_backward(Q, K, V, one, dO, 3)) < 45 * base
    base = _us(lambda: scram.sparse_attend_backward(Q, K, V, own, dO, 7))
    dO[0, H // 2, H // 2, 1] = float("nan")
    assert _us(lambda: scram.sparse_attend_backward(Q, K, V, own, dO, 7)) < 4 * base
