"""The timed cases: calls of the package's public entry points over the sizes that they serve.

Each case is one call of a layer's step -- PatchMatch maps, the sparse attend, its gradients, the
importance-sampling estimate -- or a whole forward call.  Inputs follow the recipe of
``scram_inputs`` (blurred unit-norm keys, queries that are noisy copies of coherently displaced
keys, some queries with a random target), generated on the GPU.  Calls that take maps get them as
PatchMatch leaves them: the displaced targets, a share of them a pixel or two off, a few elsewhere.
"""
import math

import numpy as np
import torch

import paper_1905_10308_amd as scram

_DEVICE = "cuda"

_DEFAULTS = dict(S=1, Hq=32, Wq=32, Hk=0, Wk=0, d=64, dtype="bf16", iters=6, window=5, kappa=1, sep=1,
                 causal=False, samples=0, radius=4, alpha=0.9, sigma=4.0, F=24.0, outliers=0.05)


def _case(op, **kw):
    c = dict(_DEFAULTS, op=op, **kw)
    c["Hk"] = c["Hk"] or c["Hq"]
    c["Wk"] = c["Wk"] or c["Wq"]
    return c


def listed():
    return [
        # the smallest forward call of the package's own workloads: launches and host time count
        _case("forward", name="forward_tiny", S=1, Hq=32, Wq=32, d=16, dtype="f32", iters=4, window=3, sigma=2.0, F=8.0,
              outliers=0.0),
        # a non-local mean over one small RGB image (three channels, the width of the paper's timing figure):
        # ragged sides, two matches, the paper's default number of sweeps
        _case("forward", name="forward_image", S=1, Hq=93, Wq=125, d=3, dtype="f32", iters=8, window=3, kappa=2, F=12.0),
        # maps of 4 x 8 heads of a 64 x 64 feature grid in 32-bit
        _case("maps", name="maps_self64", S=32, Hq=64, Wq=64, d=64, dtype="f32", iters=5, sigma=3.0, F=16.0, outliers=0.0),
        # maps of four heads of a 256 x 256 image in bf16: the package's headline workload
        _case("maps", name="maps_self256", S=4, Hq=256, Wq=256, d=64, iters=7, sigma=6.0, F=64.0),
        # two separated matches per query of an autoregressive layer, narrow heads, odd sides
        _case("maps", name="maps_causal_runs", S=8, Hq=111, Wq=97, d=32, iters=6, kappa=2, sep=2, causal=True),
        # the attend step of the headline workload
        _case("attend", name="attend_self256", S=4, Hq=256, Wq=256, d=64, window=5, sigma=6.0, F=64.0),
        # the attend step between two images of different sizes, 32-bit
        _case("attend", name="attend_cross", S=8, Hq=128, Wq=128, Hk=192, Wk=192, d=32, dtype="f32", window=3,
              outliers=0.0),
        # wide heads: attention over the union of two windows per query, odd sides
        _case("attend", name="attend_union_wide", S=8, Hq=97, Wq=111, d=128, window=5, kappa=2, sep=2),
        # the gradients of the headline workload's attend step
        _case("backward", name="backward_self256", S=4, Hq=256, Wq=256, d=64, window=5, sigma=6.0, F=64.0),
        # and those of the 32-bit heads
        _case("backward", name="backward_self64", S=32, Hq=64, Wq=64, d=64, dtype="f32", window=3, sigma=3.0, F=16.0,
              outliers=0.0),
        # the Monte Carlo estimate with its effective sample size, 32 samples per query
        _case("estimate", name="estimate_self256", S=4, Hq=256, Wq=256, d=64, samples=32, sigma=6.0, F=64.0),
        # one 2048 x 2048 image: inputs far past every cache
        _case("forward", name="forward_large", S=1, Hq=2048, Wq=2048, d=64, iters=7, window=5, sigma=6.0, F=128.0),
    ]


def draw(rng):
    op = rng.choice(["forward", "maps", "maps", "attend", "attend", "attend", "backward", "backward", "estimate"])
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))  # noqa: E731
    S, H = log(1, 32), log(32, 512)
    W = max(24, min(640, int(H * math.exp(rng.uniform(-0.5, 0.5)))))
    d = rng.choice([3, 16, 32, 64, 64, 128])
    while S * H * W * d > 1 << 25:
        S = max(1, S // 2)
        H, W = (H, W) if S > 1 else (max(32, H * 3 // 4), max(24, W * 3 // 4))
    kw = dict(S=S, Hq=H, Wq=W, d=d, dtype=rng.choice(["f32", "bf16", "bf16"]), iters=rng.randint(4, 8),
              window=rng.choice([3, 3, 5, 5, 7, 9]), sigma=rng.choice([2.0, 4.0, 6.0]), outliers=rng.choice([0.0, 0.05]))
    kw["F"] = float(min(64, max(4, min(H, W) // 5)))
    if op != "backward" and rng.random() < 0.2:  # another image as keys
        f = rng.choice([0.75, 1.5])
        kw.update(Hk=max(24, int(H * f)), Wk=max(24, int(W * f)))
    elif rng.random() < 0.25:
        kw.update(causal=True)
    if op == "estimate":
        kw.update(samples=log(8, 64))
    if rng.random() < 0.3:
        kw.update(kappa=rng.choice([2, 2, 3, 4]), sep=rng.choice([1, 2]))
    return _case(op, **kw)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _blur_matrix(n, sigma):
    """[n, n] matrix of a Gaussian blur along one axis, truncated at 4 sigma, reflecting border."""
    r = int(4.0 * sigma + 0.5)
    taps = np.exp(-0.5 * (np.arange(-r, r + 1) / sigma) ** 2)
    taps /= taps.sum()
    at = np.arange(n)[:, None] + np.arange(-r, r + 1)[None, :]
    at = np.mod(at, 2 * n)
    at = np.where(at >= n, 2 * n - 1 - at, at)
    m = np.zeros((n, n))
    np.add.at(m, (np.repeat(np.arange(n), 2 * r + 1), at.reshape(-1)), np.tile(taps, n))
    return torch.from_numpy(m.astype(np.float32)).to(_DEVICE)


def _blur(x, sigma):
    """Blur of an [H, W, c] image along both grid axes."""
    H, W, c = x.shape
    x = (_blur_matrix(H, sigma) @ x.reshape(H, W * c)).reshape(H, W, c)
    return torch.matmul(_blur_matrix(W, sigma), x)


def _inputs(c, seed):
    gen = torch.Generator(device=_DEVICE).manual_seed(int(seed))
    S, Hq, Wq, Hk, Wk, d = (c[k] for k in ("S", "Hq", "Wq", "Hk", "Wk", "d"))
    kind = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    normal = lambda *s: torch.randn(*s, generator=gen, device=_DEVICE)  # noqa: E731
    uniform = lambda *s: torch.rand(*s, generator=gen, device=_DEVICE)  # noqa: E731
    whole = lambda n, *s: torch.randint(n, s, generator=gen, device=_DEVICE)  # noqa: E731
    xs = torch.arange(Hq, device=_DEVICE)[:, None] * (Hk / Hq)
    ys = torch.arange(Wq, device=_DEVICE)[None, :] * (Wk / Wq)
    own = torch.arange(Hq * Wq, device=_DEVICE).reshape(Hq, Wq)
    K = torch.empty(S, Hk, Wk, d, dtype=kind, device=_DEVICE)
    Q = torch.empty(S, Hq, Wq, d, dtype=kind, device=_DEVICE)
    maps = torch.empty(c["kappa"], S, Hq, Wq, dtype=torch.int32, device=_DEVICE)
    eight = torch.tensor([[-1, -1], [-1, 0], [-1, 1], [0, 1], [1, 1], [1, 0], [1, -1], [0, -1]], device=_DEVICE)
    for s in range(S):
        k = _blur(normal(Hk, Wk, d), c["sigma"])
        K[s] = k / k.norm(dim=2, keepdim=True)
        f = _blur(2.0 * uniform(Hq, Wq, 2) - 1.0, 2.0 * c["sigma"])
        f = f * (c["F"] / f.norm(dim=2).max())
        tr = (xs + f[..., 0]).round().long().clamp(0, Hk - 1)
        tc = (ys + f[..., 1]).round().long().clamp(0, Wk - 1)
        if c["outliers"] > 0:
            out = uniform(Hq, Wq) < c["outliers"]
            tr = torch.where(out, whole(Hk, Hq, Wq), tr)
            tc = torch.where(out, whole(Wk, Hq, Wq), tc)
        if c["causal"]:  # the target at or before the query
            t = torch.minimum(tr * Wk + tc, own)
            tr, tc = t // Wk, t % Wk
        Q[s] = 4.0 * K[s].reshape(Hk * Wk, d).float()[(tr * Wk + tc).reshape(-1)].reshape(Hq, Wq, d) + 0.1 * normal(Hq, Wq, d)
        # matches around the target: a tenth of them a pixel or two off; further matches `sep` pixels away
        off = (uniform(Hq, Wq) < 0.1).long()
        br, bc = tr + off * (whole(5, Hq, Wq) - 2), tc + off * (whole(5, Hq, Wq) - 2)
        way = whole(8, Hq, Wq)
        for e in range(c["kappa"]):
            step = c["sep"] * eight[(way + 3 * e) % 8] if e else torch.zeros(Hq, Wq, 2, dtype=torch.long, device=_DEVICE)
            m = (br + step[..., 0]).clamp(0, Hk - 1) * Wk + (bc + step[..., 1]).clamp(0, Wk - 1)
            maps[e, s] = torch.minimum(m, own) if c["causal"] else m
    V = normal(S, Hk, Wk, d).to(kind)
    dO = normal(S, Hq, Wq, d).to(kind) if c["op"] == "backward" else None
    return Q, K, V, dO, maps if c["kappa"] > 1 else maps[0]


_PM_SEED = 12345


def prepare(case, seed):
    c = dict(case)
    c["Q"], c["K"], c["V"], c["dO"], c["maps"] = _inputs(case, seed)
    if c["op"] == "backward":  # a training loop keeps its workspace
        w = min(w for w in (16, 32, 64, 128) if w >= c["d"])  # the width that the kernels take
        need = scram.sparse_attend_backward_workspace_bytes(c["S"], c["Hq"], c["Wq"], c["Hk"], c["Wk"], c["kappa"], d=w,
                                                            dtype=c["Q"].dtype)
        c["workspace"] = torch.empty(need, dtype=torch.uint8, device=_DEVICE)
    return c


def run(state):
    c = state
    op = c["op"]
    if op == "forward":
        return scram.forward(c["Q"], c["K"], c["V"], c["iters"], _PM_SEED, c["window"], kappa=c["kappa"], sep=c["sep"],
                             causal=c["causal"])
    if op == "maps":
        if c["kappa"] == 1:
            return scram.patchmatch(c["Q"], c["K"], c["iters"], _PM_SEED, causal=c["causal"], return_score=True)
        return scram.patchmatch_kappa(c["Q"], c["K"], c["kappa"], c["iters"], _PM_SEED, sep=c["sep"], causal=c["causal"])
    if op == "attend":
        return scram.sparse_attend(c["Q"], c["K"], c["V"], c["maps"], c["window"], causal=c["causal"])
    if op == "backward":
        return scram.sparse_attend_backward(c["Q"], c["K"], c["V"], c["maps"], c["dO"], c["window"], causal=c["causal"],
                                            workspace=c["workspace"])
    out, ess, _ = scram.snis_attend(c["Q"], c["K"], c["V"], c["maps"], c["samples"], alpha=c["alpha"], radius=c["radius"],
                                    seed=_PM_SEED, causal=c["causal"], ess=True)
    return out, ess


def work(case):
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    nq, nk, d, kappa = c["S"] * c["Hq"] * c["Wq"], c["S"] * c["Hk"] * c["Wk"], c["d"], c["kappa"]
    q, k, maps = nq * d * e, nk * d * e, kappa * nq * 4
    candidates = 16 + int(math.log2(max(c["Hk"], c["Wk"]))) + 1
    keys = kappa * c["window"] ** 2
    search = 2 * d * candidates * c["iters"] * nq * kappa
    if c["op"] == "forward":
        return {"bytes": 2 * q + 2 * k + maps, "flops": search + 4 * d * keys * nq}
    if c["op"] == "maps":
        return {"bytes": q + k + maps + (4 * nq if kappa == 1 else 0), "flops": search}
    if c["op"] == "attend":
        return {"bytes": 2 * q + 2 * k + maps, "flops": 4 * d * keys * nq}
    if c["op"] == "backward":
        return {"bytes": 2 * q + 2 * k + maps + 4 * d * nq + 8 * d * nk, "flops": 10 * d * keys * nq}
    return {"bytes": 2 * q + 2 * k + maps + 4 * nq, "flops": 4 * d * c["samples"] * nq}


def tolerance(case):
    """About four times the largest difference from `exact` seen over the listed and some drawn cases."""
    if case["op"] == "maps":
        # a decision between two keys whose scores differ by less than the 32-bit sums resolve may go either way,
        # and moves what propagates from it: up to 1e-4 of the entries, their scores by up to 9e-7 (5e-4 at most)
        return {"rel": 4e-6, "max": 2e-3, "differ": 5e-4}
    if case["op"] == "forward":
        # such a decision also moves a whole output row; with three channels 2e-4 of the rows, 1.4e-2 in all
        return {"rel": 2e-2, "max": 0.99, "differ": 1e-3}
    if case["op"] == "backward":  # 32-bit gradients of either storage type: 6e-7, 2.5e-5 at most
        return {"rel": 3e-6, "max": 1e-4}
    if case["dtype"] == "bf16":  # the rounding of the output: 1.7e-3, 2^-8 at most
        return {"rel": 7e-3, "max": 1.6e-2}
    return {"rel": 8e-7, "max": 5e-6}


# ---------------------------------------------------------------------------
# the same results in 64 bits, in plain torch
# ---------------------------------------------------------------------------
def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 of int64 tensors (or numbers) holding 32-bit words."""
    m32 = 0xFFFFFFFF
    k0, k1 = seed & m32, (seed >> 32) & m32
    for _ in range(10):
        a, b = c0 * 0xD2511F53, c2 * 0xCD9E8D57  # wrapped to 64 bits; the shift is masked below
        c0, c1, c2, c3 = ((b >> 32) & m32) ^ c1 ^ k0, b & m32, ((a >> 32) & m32) ^ c3 ^ k1, a & m32
        k0, k1 = (k0 + 0x9E3779B9) & m32, (k1 + 0xBB67AE85) & m32
    return c0, c1, c2, c3


def _patchmatch64(c, Q, K, prev):
    """Maps [S * Hq * Wq] and their scores after c["iters"] synchronous sweeps, given the earlier runs' maps."""
    S, Hq, Wq, Hk, Wk, d = (c[k] for k in ("S", "Hq", "Wq", "Hk", "Wk", "d"))
    n, run = S * Hq * Wq, len(prev)
    g = torch.arange(n, device=_DEVICE)
    s, rem = g // (Hq * Wq), g % (Hq * Wq)
    x, y = rem // Wq, rem % Wq
    Qf, Kf = Q.reshape(n, d), K.reshape(S * Hk * Wk, d)

    def score(j):
        got = torch.empty(n, dtype=torch.float64, device=_DEVICE)
        for b in range(0, n, 1 << 20):
            e = min(n, b + (1 << 20))
            got[b:e] = (Qf[b:e].double() * Kf[(s * Hk * Wk + j)[b:e]].double()).sum(1)
        return got

    def valid(u, v):
        ok = (u * Wk + v <= rem) if c["causal"] else torch.ones(n, dtype=torch.bool, device=_DEVICE)
        for m in prev:
            ok = ok & (torch.maximum((u - m // Wk).abs(), (v - m % Wk).abs()) >= c["sep"])
        return ok

    g32 = g & 0xFFFFFFFF
    w = _philox(g32, torch.zeros_like(g), torch.zeros_like(g), torch.full_like(g, run), _PM_SEED)
    J = (w[0] * (rem + 1)) >> 32 if c["causal"] else ((w[0] * Hk) >> 32) * Wk + ((w[1] * Wk) >> 32)
    best = score(J)
    for t in range(1, c["iters"] + 1):
        best = torch.where(valid(J // Wk, J % Wk), best, torch.full_like(best, -math.inf))
        cur, old = J.clone(), J.reshape(S, Hq, Wq)

        def consider(u, v, ok):
            ok = ok & valid(u, v)
            j = torch.where(ok, u * Wk + v, cur)
            sc = score(j)
            take = ok & ((sc > best) | ((sc == best) & (j < cur)))
            return torch.where(take, j, cur), torch.where(take, sc, best)

        for jump in (8, 4, 2, 1):
            for ox, oy in ((-jump, 0), (jump, 0), (0, -jump), (0, jump)):
                nx, ny = x + ox, y + oy
                ok = (nx >= 0) & (nx < Hq) & (ny >= 0) & (ny < Wq)
                nb = old[s, nx.clamp(0, Hq - 1), ny.clamp(0, Wq - 1)]
                u, v = nb // Wk - ox, nb % Wk - oy
                ok = ok & (u >= 0) & (u < Hk) & (v >= 0) & (v < Wk)
                cur, best = consider(u, v, ok)
        D, k = max(Hk, Wk), 0
        while D >= 1:
            w = _philox(g32, torch.full_like(g, t), torch.full_like(g, k // 2), torch.full_like(g, run), _PM_SEED)
            u, v = cur // Wk, cur % Wk
            lr, hr = (u - D).clamp(min=0), (u + D).clamp(max=Hk - 1)
            lc, hc = (v - D).clamp(min=0), (v + D).clamp(max=Wk - 1)
            r = lr + ((w[2 * (k % 2)] * (hr - lr + 1)) >> 32)
            q = lc + ((w[2 * (k % 2) + 1] * (hc - lc + 1)) >> 32)
            cur, best = consider(r, q, torch.ones(n, dtype=torch.bool, device=_DEVICE))
            D, k = D // 2, k + 1
        J = cur
    return J, best


def _key_slots(c, maps, b, e):
    """For each key slot of the union of the windows of queries b .. e - 1: (flat key in the slice, whether it counts)."""
    Hk, Wk, half = c["Hk"], c["Wk"], c["window"] // 2
    rem = torch.arange(b, e, device=_DEVICE) % (c["Hq"] * c["Wq"])
    u0, v0 = [m[b:e] // Wk for m in maps], [m[b:e] % Wk for m in maps]
    got = []
    for i, m in enumerate(maps):
        for a in range(-half, half + 1):
            for o in range(-half, half + 1):
                u, v = u0[i] + a, v0[i] + o
                ok = (u >= 0) & (u < Hk) & (v >= 0) & (v < Wk)
                for f in range(i):
                    ok = ok & ~(((u - u0[f]).abs() <= half) & ((v - v0[f]).abs() <= half))
                if c["causal"]:
                    ok = ok & (u * Wk + v <= rem)
                got.append((torch.where(ok, u * Wk + v, m[b:e]), ok))
    return got


def _attend64(c, Q, K, V, maps, dO=None):
    """The softmax over each query's windows times the values; with dO the gradients (dQ, dK, dV) instead."""
    S, Hq, Wq, Hk, Wk, d = (c[k] for k in ("S", "Hq", "Wq", "Hk", "Wk", "d"))
    n, nk, scale = S * Hq * Wq, Hk * Wk, d ** -0.5
    zeros = lambda m: torch.zeros(m, d, dtype=torch.float64, device=_DEVICE)  # noqa: E731
    Qf, Kf, Vf = Q.reshape(n, d), K.reshape(S * nk, d), V.reshape(S * nk, d)
    out, dK, dV = zeros(n), zeros(S * nk if dO is not None else 0), zeros(S * nk if dO is not None else 0)
    for b in range(0, n, 1 << 18):
        e = min(n, b + (1 << 18))
        base = torch.arange(b, e, device=_DEVICE) // (Hq * Wq) * nk
        slots = _key_slots(c, maps, b, e)
        q = Qf[b:e].double()
        sc = torch.stack([torch.where(ok, scale * (q * Kf[base + j].double()).sum(1), -math.inf) for j, ok in slots])
        p = torch.softmax(sc, 0).nan_to_num(0.0)  # no key at all: a zero row
        if dO is None:
            for w, (j, _) in zip(p, slots):
                out[b:e] += w[:, None] * Vf[base + j].double()
            continue
        do = dO.reshape(n, d)[b:e].double()
        dp = torch.stack([(do * Vf[base + j].double()).sum(1) for j, _ in slots])
        ds = scale * p * (dp - (p * dp).sum(0))
        for w, dw, (j, _) in zip(p, ds, slots):
            out[b:e] += dw[:, None] * Kf[base + j].double()
            dK.index_add_(0, base + j, dw[:, None] * q)
            dV.index_add_(0, base + j, w[:, None] * do)
    out = out.reshape(S, Hq, Wq, d)
    return out if dO is None else (out, dK.reshape(S, Hk, Wk, d), dV.reshape(S, Hk, Wk, d))


def _estimate64(c, Q, K, V, maps):
    """The self-normalised importance-sampling estimate and its effective sample size."""
    S, Hq, Wq, Hk, Wk, d, T, m = (c[k] for k in ("S", "Hq", "Wq", "Hk", "Wk", "d", "samples", "radius"))
    n, nk, kappa, scale = S * Hq * Wq, Hk * Wk, len(maps), d ** -0.5
    g = torch.arange(n, device=_DEVICE)
    base, rem = g // (Hq * Wq) * nk, g % (Hq * Wq)
    Qd, Kf, Vf = Q.reshape(n, d).double(), K.reshape(S * nk, d), V.reshape(S * nk, d)
    alpha16 = math.floor(c["alpha"] * 65536 + 0.5)
    alpha = alpha16 / 65536
    pmf = torch.tensor([math.comb(2 * m, i) / 4.0 ** m for i in range(2 * m + 1)], dtype=torch.float64, device=_DEVICE)
    cdf = pmf.cumsum(0)
    cu, cv = torch.stack([j // Wk for j in maps]), torch.stack([j % Wk for j in maps])

    def bits(w):
        w = w & ((1 << (2 * m)) - 1)
        return sum((w >> i) & 1 for i in range(2 * m)) - m

    def axis(r, centre, size):
        def tail(x):
            return torch.where(x < -m, 0.0, torch.where(x >= m, 1.0, cdf[(x + m).clamp(0, 2 * m)]))

        x = r - centre
        inside = torch.where(x.abs() <= m, pmf[(x + m).clamp(0, 2 * m)], 0.0)
        edge = torch.where(r == 0, tail(-centre), tail(centre - (size - 1)))
        return torch.where((r == 0) | (r == size - 1), edge, inside)

    keys, logw = [], []
    for t in range(T):
        w = _philox(g & 0xFFFFFFFF, torch.full_like(g, t), torch.zeros_like(g), torch.full_like(g, 0x534E4953), _PM_SEED)
        e = ((w[1] * kappa) >> 32)[None]
        near = (w[0] >> 16) < alpha16
        r = torch.where(near, (cu.gather(0, e)[0] + bits(w[2])).clamp(0, Hk - 1), (w[2] * Hk) >> 32)
        q = torch.where(near, (cv.gather(0, e)[0] + bits(w[3])).clamp(0, Wk - 1), (w[3] * Wk) >> 32)
        local = sum(axis(r, cu[f], Hk) * axis(q, cv[f], Wk) for f in range(kappa))
        j = r * Wk + q
        a = scale * (Qd * Kf[base + j].double()).sum(1) - (alpha / kappa * local + (1 - alpha) / nk).log()
        keys.append(j)
        logw.append(torch.where(j > rem, -math.inf, a) if c["causal"] else a)
    lw = torch.stack(logw)
    wt = (lw - lw.max(0).values).exp().nan_to_num(0.0)
    total = wt.sum(0)
    out = torch.zeros(n, d, dtype=torch.float64, device=_DEVICE)
    for w, j in zip(wt, keys):
        out += (w / total.clamp(min=1e-300))[:, None] * Vf[base + j].double()
    ess = torch.where(total > 0, total.square() / wt.square().sum(0).clamp(min=1e-300), 0.0)
    return out.reshape(S, Hq, Wq, d), ess.reshape(S, Hq, Wq)


def exact(case, seed):
    c = case
    Q, K, V, dO, maps = _inputs(c, seed)
    shape = (c["S"], c["Hq"], c["Wq"])
    if c["op"] in ("forward", "maps"):
        runs, score = [], None
        for _ in range(c["kappa"]):
            J, score = _patchmatch64(c, Q, K, runs)
            runs.append(J)
        J = torch.stack(runs).reshape(c["kappa"], *shape).int()
        if c["op"] == "forward":
            return _attend64(c, Q, K, V, runs), J
        return (J[0], score.reshape(shape)) if c["kappa"] == 1 else J
    maps = [m.reshape(-1).long() for m in (maps if c["kappa"] > 1 else maps[None])]
    if c["op"] == "attend":
        return _attend64(c, Q, K, V, maps)
    if c["op"] == "backward":
        return _attend64(c, Q, K, V, maps, dO)
    return _estimate64(c, Q, K, V, maps)
