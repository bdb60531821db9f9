"""The matrix-core attend at 16 and 128 channels and with 9 x 9 windows, against the oracle (``-m gpu``)."""
import numpy as np
import pytest
import torch

import oracle
import scram_inputs.synth as synth
from gpu_util import TOL, row_rel_err, tile_maps, to_dev

pytestmark = pytest.mark.gpu

# 16 and 128 channels take the matrix cores from 7 x 7 on, 128 also with several 5 x 5 windows, 32 and 64 with 9 x 9 too;
# (16, 5), (128, 3) and (128, 5) with one map take the lane-group kernels: controls
SHAPES = [(16, 5), (16, 7), (16, 9), (32, 9), (64, 9), (128, 3), (128, 5), (128, 7), (128, 9)]
# several tiles with ragged edges, the smallest grids, one row, one column, two grids, and a grid on which a wave's
# random matches lie too far apart for the matrix cores
GRIDS = [(2, 21, 37, 21, 37), (1, 3, 5, 3, 5), (1, 1, 50, 1, 50), (1, 50, 1, 50, 1), (1, 19, 11, 33, 30),
         (1, 40, 61, 40, 61)]


def attend(scram, Q, K, V, J, window, scale=None, causal=False):
    """``sparse_attend`` of slices in numpy; with 128 channels of 512 copies of them, so that the call is wide enough
    for the matrix cores, every copy with the same bits."""
    n, S = (512 if Q.shape[-1] == 128 else 1), Q.shape[0]
    dev = [to_dev(x, "bf16").repeat(n, 1, 1, 1) for x in (Q, K, V)]
    Jd = torch.from_numpy(np.ascontiguousarray(J)).cuda().repeat(1, n, 1, 1)
    got = scram.sparse_attend(*dev, Jd, window, scale, causal=causal)
    assert (got.view(torch.int16).reshape(n, -1) == got[:S].view(torch.int16).reshape(1, -1)).all()
    return got[:S]


@pytest.mark.parametrize("d,window", SHAPES)
@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
def test_attend_widths(scram, d, window, grid):
    S, Hq, Wq, Hk, Wk = grid
    rng = np.random.default_rng(d + window + Hq)
    Q, K, V = (synth._round_bf16(rng.standard_normal(s).astype(np.float32)) for s in
               ((S, Hq, Wq, d), (S, Hk, Wk, d), (S, Hk, Wk, d)))
    m = tile_maps(S, Hq, Wq, Hk, Wk, rng)
    sets = [m[n][None] for n in ("random", "coherent", "lattice7", "lattice10", "two_far", "outliers")]
    sets += [np.stack([m["coherent"], m["outliers"]]), np.stack([m["random"], m["coherent"], m["corner_last"]])]
    for J in sets:
        for causal in ((False, True) if (Hq, Wq) == (Hk, Wk) else (False,)):
            got = attend(scram, Q, K, V, J, window, causal=causal)
            ref = oracle.sparse_attend(Q, K, V, J, window, d ** -0.5, flags=oracle.CAUSAL if causal else 0)
            err = row_rel_err(got.double().cpu().numpy(), ref)
            assert err.max() <= TOL["bf16"], (J.shape[0], causal, err.max())
            empty = ~np.any(ref, axis=-1)
            assert not got.cpu()[torch.from_numpy(empty)].any()  # a query without keys: a zero row


@pytest.mark.parametrize("d,window", SHAPES)
def test_non_finite_values_stay_in_their_windows(scram, d, window):
    """A value row with an infinity or a NaN reaches exactly the queries whose windows hold its key, although
    the rows are read in blocks that neighbouring queries share."""
    S, H, W, b = 1, 24, 24, window // 2
    rng = np.random.default_rng(d + window)
    Q, K, V = (synth._round_bf16(rng.standard_normal((S, H, W, d)).astype(np.float32)) for _ in range(3))
    J = np.stack([np.arange(H * W).reshape(S, H, W), rng.integers(0, H * W, (S, H, W))]).astype(np.int32)
    clean = attend(scram, Q, K, V, J, window)
    bad = [(7, 9), (20, 3)]
    V[0, 7, 9, d // 2] = np.inf
    V[0, 20, 3, 1] = np.nan
    got = attend(scram, Q, K, V, J, window)
    near = np.zeros((S, H, W), bool)
    for u, v in bad:
        for m in J:
            near |= (np.abs(m // W - u) <= b) & (np.abs(m % W - v) <= b)
    got, clean = got.float().cpu().numpy(), clean.float().cpu().numpy()
    assert np.isfinite(got[~near]).all()
    np.testing.assert_allclose(got[~near], clean[~near], rtol=2 ** -7, atol=1e-3)  # (bf16 rounding of either path)
    assert (~np.isfinite(got[near])).any(axis=-1).all()


def key_sets(J, H, W, window, causal):
    """[queries, keys] of one slice: whether the union of the query's windows holds the key."""
    b, n = window // 2, H * W
    k = np.arange(n)
    held = np.zeros((n, n), bool)
    for m in J.reshape(len(J), n):
        held |= (np.abs(m[:, None] // W - k[None] // W) <= b) & (np.abs(m[:, None] % W - k[None] % W) <= b)
    return held & (k[None] <= k[:, None]) if causal else held


def unit_case(d, kappa, seed):
    """Keys, values, queries and maps on one 24 x 24 grid: the queries' own keys, scattered ones, shifted ones."""
    H = W = 24
    rng = np.random.default_rng(seed)
    Q, K, V = (synth._round_bf16(rng.standard_normal((1, H, W, d)).astype(np.float32)) for _ in range(3))
    own = np.arange(H * W).reshape(1, H, W)
    J = np.stack([own, rng.integers(0, H * W, (1, H, W)), np.roll(own, 5, 2)][:kappa]).astype(np.int32)
    return H, W, Q, K, V, J


@pytest.mark.parametrize("d,window", SHAPES)
@pytest.mark.parametrize("kappa", [1, 2, 3])
@pytest.mark.parametrize("causal", [False, True])
def test_non_finite_values_stay_in_their_channels(scram, d, window, kappa, causal):
    """Of a query whose set holds a value row with an infinity or a NaN in one channel, that channel is not
    finite and every other one holds what it held: a row has one writer."""
    H, W, Q, K, V, J = unit_case(d, kappa, d + window + kappa)
    clean = attend(scram, Q, K, V, J, window, causal=causal).float().cpu().numpy().reshape(H * W, d)
    bad = {7 * W + 9: (d // 2, np.inf), 3 * W + 3: (1, np.nan), 12 * W + 20: (d - 1, -np.inf)}
    for k, (ch, x) in bad.items():
        V[0, k // W, k % W, ch] = x
    got = attend(scram, Q, K, V, J, window, causal=causal)
    got = got.float().cpu().numpy().reshape(H * W, d)
    held = key_sets(J, H, W, window, causal)
    off = np.zeros((H * W, d), bool)
    for k, (ch, _) in bad.items():
        off[held[:, k], ch] = True
    assert off.any()
    if causal and (window == 3 or (window == 5 and (d == 16 or kappa == 1))):
        # the lane-group kernels: a key that the mask drops from a window row of the set may reach it through 0 * inf
        for k, (ch, _) in bad.items():
            off[key_sets(J, H, W, window, False)[:, k] & ~np.isfinite(got[:, ch]), ch] = True
    np.testing.assert_array_equal(~np.isfinite(got), off)
    np.testing.assert_allclose(got[~off], clean[~off], rtol=2 ** -7, atol=1e-3)  # (bf16 rounding of either path)


def attend_by_batches(q, K, V, J, i, H, W, window, scale, causal):
    """Query i's row in fp64 (K, V: [keys, d]; J: [kappa, queries]) as the lane-group kernels define it for scores
    that are not finite: the reference is raised a batch of keys at a time (a window row; 4 slots of windows above
    7 x 7), and a batch without a score that is a number is left out while there is no reference."""
    b, kept, seen, poisoned, ref = window // 2, [], set(), False, -np.inf
    for m in J[:, i]:
        u, v = divmod(int(m), W)
        rows = [[r * W + c for c in range(max(v - b, 0), min(v + b, W - 1) + 1)]
                for r in range(max(u - b, 0), min(u + b, H - 1) + 1)]
        slots = sum(rows, [])
        batches = rows if window <= 7 else [slots[k:k + 4] for k in range(0, len(slots), 4)]
        for batch in batches:
            keys = [k for k in batch if k not in seen and not (causal and k > i)]
            if not keys:
                continue
            sc = K[keys] @ q * scale
            ref = max([ref, *sc[~np.isnan(sc)]])
            if ref == -np.inf:
                continue
            poisoned |= bool(np.isnan(sc).any() or ref == np.inf)
            kept += [(k, x) for k, x in zip(keys, sc) if x > -np.inf]
        seen |= set(slots)
    if poisoned:
        return np.full(V.shape[1], np.nan)
    if not kept:
        return np.zeros(V.shape[1])
    w = np.exp(np.array([x for _, x in kept]) - max(x for _, x in kept))
    return (w / w.sum()) @ V[[k for k, _ in kept]]


@pytest.mark.parametrize("d,window", SHAPES)
@pytest.mark.parametrize("kappa", [1, 2, 3])
@pytest.mark.parametrize("causal", [False, True])
def test_scores_that_are_not_finite(scram, d, window, kappa, causal):
    """A key row with a NaN (every score of the key is NaN) or an infinity (scores of either sign) counts wherever
    it lies in a window -- its first key, its last, one between -- and not outside; a query of NaNs has no score."""
    H, W, Q, K, V, J = unit_case(d, kappa, 3 * d + window + kappa)
    K[0, 0, 0, 1] = K[0, 9, 13, d - 1] = np.nan
    K[0, 15, 6, d // 2] = np.inf
    Q[0, 20, 20] = np.nan
    got = attend(scram, Q, K, V, J, window, causal=causal)
    got = got.double().cpu().numpy().reshape(H * W, d)
    Qf, Kf, Vf = (x.astype(np.float64).reshape(H * W, d) for x in (Q, K, V))
    with np.errstate(invalid="ignore"):
        ref = np.stack([attend_by_batches(Qf[i], Kf, Vf, J.reshape(kappa, -1), i, H, W, window, d ** -0.5, causal)
                        for i in range(H * W)])
    nan = np.isnan(ref).any(1)
    assert nan.any() and not nan.all()
    np.testing.assert_array_equal(np.isnan(got).all(1), nan)
    assert np.isfinite(got[~nan]).all()
    assert row_rel_err(got[~nan], ref[~nan]).max() <= TOL["bf16"]


@pytest.mark.parametrize("d,window", SHAPES)
@pytest.mark.parametrize("kappa", [1, 2])
def test_weights_keep_24_bits(scram, d, window, kappa):
    """Windows of three keys that count (scores 0, 0, x; the others' weights underflow to 0) with values -hi, -mid and
    1, where hi and mid are the first and the second 8 significant bits of w = 2^x: the row is (w - hi - mid) / (2 + w),
    the last 8 bits of w, and zero or worse where a weight holds 16 bits.  Bound: 2^x, its exponent's rounding and
    the three sums err by at most 4 units of w's last place, the output by 2^-8 of itself."""
    step, n = window + 1, 4
    H = W = step * n
    scale = 2.0 ** -3
    per = scale * 1.4426950408889634  # log2 of a weight per unit of the score q . k
    x = -np.arange(1, n * n + 1) / 16 - 0.03125
    score = synth._round_bf16((x / per).astype(np.float32)).astype(np.float64)
    w = np.exp2(score * per)  # (0.5, 1) and below: 24 bits
    ulp = np.exp2(np.floor(np.log2(w)) - 23)

    def cut(a):  # the top 8 significant bits
        return (a.astype(np.float32).view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32).astype(np.float64)

    hi = cut(w)
    mid = cut(w - hi)
    want = (w - hi - mid) / (2 + w)
    K, V = (np.zeros((1, H, W, d), np.float32) for _ in range(2))
    K[..., 0] = -4096.0  # a weight of 2^-738: 0
    centre = np.zeros(n * n, np.int64)
    for t in range(n * n):
        u, v = (t // n) * step + step // 2, (t % n) * step + step // 2
        centre[t] = u * W + v
        for c, (s, val) in enumerate([(0.0, -hi[t]), (0.0, -mid[t]), (score[t], 1.0)]):
            K[0, u, v + c - 1, 0] = s
            V[0, u, v + c - 1] = val
    Q = np.zeros((1, H, W, d), np.float32)
    Q[..., 0] = 1.0
    t = np.arange(H * W) % (n * n)
    J = np.broadcast_to(centre[t].reshape(1, 1, H, W), (kappa, 1, H, W)).astype(np.int32)
    for a in (Q, K, V):
        assert np.array_equal(synth._round_bf16(a), a)  # (exact in bf16)
    got = attend(scram, Q, K, V, J, window, scale)
    got = got.double().cpu().numpy().reshape(H * W, d)
    sharp = (want > 32 * ulp)[t]
    assert sharp.sum() >= H * W // 4
    err = np.abs(got - want[t][:, None])
    assert (err <= (4 * ulp / (2 + w) + 2.0 ** -8 * want)[t][:, None])[sharp].all(), err[sharp].max()
