"""The work that programs have this library do, as cases with sizes.

A case is one call, or the few calls that belong together, of a program that
factorises a rating matrix on one GPU: a training run that ends with the factors
in host memory, the float64 variant, element-wise CCD, a whole fit from host
triplets, training watched on a held-out set, the held-out RMSE of a trained
model, and training resumed from saved factors.  The shapes are the workloads
that paper_1511_02433_amd.synth declares and sizes between them.

Every input is drawn from the seed on the GPU: a rating matrix whose users and
items have power-law degrees (a shifted rank curve, density (r + count / 200)^-a
over the ranks r), ids in no order of degree, ratings 1..5 from a latent score
plus noise, triplets grouped by user as rating files are.
"""
import math

import numpy as np
import torch

from paper_1511_02433_amd.ccdpp import CCDPP, make_options

SIDES = {
    # uniform-like small matrix of the quick tests
    "tiny": dict(m=2_000, n=1_000, nnz=50_000, lam=0.05, au=0.0, ai=0.0),
    # a million ratings: what a first experiment holds
    "small": dict(m=6_041, n=3_707, nnz=1_000_209, lam=0.05, au=1.001, ai=1.001),
    # ten million ratings
    "medium": dict(m=71_567, n=10_681, nnz=10_000_054, lam=0.05, au=1.2, ai=1.2),
    # many users and items with about twenty ratings each: a sparse catalogue
    "sparse": dict(m=300_007, n=150_001, nnz=6_000_011, lam=1.0, au=1.001, ai=1.1),
    # the paper's matrix (Section 8): 100.5M ratings
    "large": dict(m=480_189, n=17_770, nnz=100_480_507, lam=0.05, au=1.1, ai=0.9),
    # 252.8M ratings, both sides long
    "vlarge": dict(m=1_000_990, n=624_961, nnz=252_800_275, lam=1.0, au=1.001, ai=1.3),
}


def _case(name, kind, side, k, outer, inner, f64=False, held=0):
    return dict(SIDES[side], name=name, kind=kind, k=k, outer=outer, inner=inner, f64=f64, held=held)


def listed():
    return [
        # Training: outer x inner iterations on a handle that a program keeps, then the factors.
        # The smallest: latency and launches count.
        _case("train_tiny", "train", "tiny", 8, 5, 3),
        # A million ratings, the size of a quick experiment or of one cell of a parameter search.
        _case("train_small", "train", "small", 20, 5, 3),
        # Ten million ratings at the usual rank.
        _case("train_medium", "train", "medium", 40, 2, 3),
        # The same matrix in the paper's double version.
        _case("train_medium_f64", "train", "medium", 20, 2, 2, f64=True),
        # Sparse rows on both sides, one inner iteration.
        _case("train_sparse", "train", "sparse", 16, 2, 1),
        # The paper's matrix at the first rank of the rank sweep (5 x 3).
        _case("train_large", "train", "large", 10, 5, 3),
        # The largest matrix.
        _case("train_vlarge", "train", "vlarge", 4, 2, 3),
        # Element-wise CCD (Algorithm 2).
        _case("ccd_medium", "ccd", "medium", 20, 2, 1),
        # Everything from the host's triplets to the host's factors: build, train, copy out, free.
        _case("fit_medium", "fit", "medium", 40, 3, 3),
        # Training with the objective and the held-out RMSE after every outer iteration.
        _case("monitor_medium", "monitor", "medium", 40, 2, 3, held=200_003),
        # The held-out RMSE of a trained model, as after each change of a setting.
        _case("evaluate_large", "evaluate", "large", 40, 0, 1, held=1_400_000),
        # A saved model goes on: its factors set, one more outer iteration, the factors out.
        _case("resume_large", "resume", "large", 40, 1, 3),
    ]


def draw(rng):
    kind = rng.choice(["train"] * 6 + ["ccd", "fit", "monitor", "evaluate", "resume", "resume"])
    nnz = int(round(math.exp(rng.uniform(math.log(50_000), math.log(60_000_000)))))
    n = int(min(400_000, max(250, nnz / math.exp(rng.uniform(math.log(12), math.log(4000))))))
    m = int(min(1_000_000, max(500, nnz / math.exp(rng.uniform(math.log(12), math.log(700))))))
    m = max(m, 20 * nnz // n + 1)  # at most a twentieth of the positions hold a rating
    k = int(round(math.exp(rng.uniform(math.log(3), math.log(64)))))
    inner = 1 if kind == "ccd" else rng.choice([1, 2, 3, 3])
    outer = {"evaluate": 0, "resume": 1}.get(kind, rng.randint(1, 5))
    k = max(2, min(k, int(12e9 / (nnz * max(outer, 1) * inner))))
    return dict(kind=kind, m=m, n=n, nnz=nnz, lam=rng.choice([0.05, 0.2, 1.0]) if nnz >= 30 * max(m, n) else 1.0,
                au=rng.choice([0.9, 1.001, 1.1, 1.2]), ai=rng.choice([0.9, 1.001, 1.1, 1.3]), k=k, outer=outer, inner=inner,
                f64=kind in ("train", "ccd", "evaluate") and rng.random() < 0.25,
                held=int(min(1_500_000, max(1_000, nnz // 50))) if kind in ("monitor", "evaluate") else 0)


# ---- inputs ------------------------------------------------------------------------


def _ids(gen, count, size, a):
    """`size` ids below count, id popularity a power law of exponent a over a fixed scramble of the ids."""
    x = torch.rand(size, generator=gen, device="cuda", dtype=torch.float64)
    if a == 0.0:
        r = x * count
    else:
        r0 = count / 200.0
        lo, hi = r0 ** (1.0 - a), (count + r0) ** (1.0 - a)
        r = (lo + x * (hi - lo)) ** (1.0 / (1.0 - a)) - r0
    r = r.to(torch.int64).clamp_(0, count - 1)
    step = int(count * 0.6180339887) | 1
    while math.gcd(step, count) != 1:
        step += 2
    return (r * step + count // 3) % count


def _triplets(case, seed):
    """(row, col, val) of the ratings and of the held-out set, on the GPU, grouped by row."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    m, n, want = case["m"], case["n"], case["nnz"] + case["held"]
    keys = torch.empty(0, dtype=torch.int64, device="cuda")
    while keys.numel() < want:
        more = int((want - keys.numel()) * 1.3) + 1000
        new = _ids(gen, m, more, case["au"]) * n + _ids(gen, n, more, case["ai"])
        keys = torch.unique(torch.cat([keys, new]) if keys.numel() else new)
        del new
    have = keys.numel()
    # What is too many, and then the held-out entries, at even distances.
    for drop in (have - want, case["held"]):
        at = torch.arange(drop, device="cuda") * keys.numel() // max(drop, 1)
        keep = torch.ones(keys.numel(), dtype=torch.bool, device="cuda")
        keep[at] = False
        held, keys = keys[at], keys[keep]
    x = torch.randn(m, 4, generator=gen, device="cuda")
    y = torch.randn(n, 4, generator=gen, device="cuda")
    out = []
    for part in (keys, held):
        row, col = (part // n).to(torch.int32), (part % n).to(torch.int32)
        val = torch.empty(part.numel(), device="cuda")
        for s in range(0, part.numel(), 1 << 24):
            e = min(part.numel(), s + (1 << 24))
            z = (x[row[s:e].long()] * y[col[s:e].long()]).sum(1) * 0.5
            val[s:e] = (3.6 + z + 0.8 * torch.randn(e - s, generator=gen, device="cuda")).round_().clamp_(1.0, 5.0)
        out.append((row, col, val))
    return out


def _factors(case, seed):
    """Row-major float32 factors: of a model part-way through its training (W, H), or the initial H, N(0, 0.01)."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed) + 77)
    k = case["k"]
    h0 = torch.randn(case["n"], k, generator=gen, device="cuda") * 0.1
    if case["kind"] in ("train", "ccd", "fit", "monitor"):
        return None, h0
    fade = 1.0 / torch.arange(1, k + 1, device="cuda").sqrt()
    w = torch.randn(case["m"], k, generator=gen, device="cuda") * 0.5 * fade
    h = torch.randn(case["n"], k, generator=gen, device="cuda") * 0.5 * fade
    w[:, 0] += 2.0
    h[:, 0] += 1.6
    return w, h


def _host(t):
    return t.cpu().numpy()


def prepare(case, seed):
    train, held = _triplets(case, seed)
    arrays = tuple(_host(x) for x in train)
    state = {"case": case, "seed": int(seed) % (1 << 62), "held": tuple(_host(x) for x in held)}
    w, h = _factors(case, seed)
    del train, held
    if case["kind"] == "fit":
        state["triplets"] = arrays
        return state
    opts = make_options(precision=1 if case["f64"] else 0)
    model = CCDPP(case["m"], case["n"], case["k"], case["lam"], *arrays, seed=1, opts=opts)
    if case["kind"] == "resume":
        state["saved"] = (_host(w), _host(h))
    elif case["kind"] == "evaluate":
        model.set_factors(_host(w), _host(h))
    else:
        model.set_factors(None, _host(h))
    state["model"] = model
    return state


def run(state):
    case, kind = state["case"], state["case"]["kind"]
    if kind == "fit":
        with CCDPP(case["m"], case["n"], case["k"], case["lam"], *state["triplets"], seed=state["seed"]) as model:
            model.run(case["outer"], case["inner"])
            return model.factors()
    model = state["model"]
    if kind == "evaluate":
        return model.rmse(*state["held"])
    if kind == "monitor":
        _, history = model.run_until(case["outer"], case["inner"], -1.0, state["held"])
        return (history,) + model.factors()
    if kind == "ccd":
        model.ccd_run(case["outer"])
    else:
        if kind == "resume":
            model.set_factors(*state["saved"])
        model.run(case["outer"], case["inner"])
    return model.factors_f64() if case["f64"] else model.factors()


# ---- what a pass needs, and what it gives --------------------------------------------


def work(case):
    """Per feature and outer iteration, CCD++ reads every rating's residual and the
    position of the other side 2 * inner times (once by user and once by item for each
    inner iteration) and writes the residual back twice; element-wise CCD reads and
    writes it once in each of its two phases.  A position is 2 bytes, or 4 where the
    other side has more than 65,536 ids.  Fit adds the host's triplets, the held-out
    RMSE its triplets and their rows of W and H, resuming the rebuilt residual."""
    m, n, k, nnz = case["m"], case["n"], case["k"], case["nnz"]
    vb = 8 if case["f64"] else 4
    pu, pi = 2 if n <= 65536 else 4, 2 if m <= 65536 else 4
    reads = 1 if case["kind"] == "ccd" else case["inner"]
    sweep = case["outer"] * k * nnz * (reads * (2 * vb + pu + pi) + 2 * vb)
    factors = (m + n) * k * vb
    held = case["held"] * (12 + 2 * k * vb)
    out = {"bytes": sweep + factors, "flops": case["outer"] * k * nnz * (2 * reads * 4 + 8)}
    if case["kind"] == "fit":
        out["bytes"] += 12 * nnz
    elif case["kind"] == "monitor":
        out["bytes"] += case["outer"] * held
    elif case["kind"] == "resume":
        out["bytes"] += factors + nnz * (2 * vb + pu)
        out["flops"] += 2 * k * nnz
    elif case["kind"] == "evaluate":
        out = {"bytes": min(held, case["held"] * 12 + factors), "flops": 2 * k * case["held"]}
    return out


def tolerance(case):
    """About four times what the sums in another order (other shares per workgroup, other
    segment weights) change after two passes on one handle, over the listed cases and
    fourteen drawn ones: float32 training 2.6e-6 (largest value 4.9e-4), float64 1.3e-15
    (1.7e-14) on ten million ratings, small matrices more."""
    if case["kind"] == "evaluate":
        return {"rel": 1e-12}  # float64 sums of the same products, in any order
    if case["f64"]:
        return {"rel": 1e-12, "max": 1e-10}
    return {"rel": 1e-5, "max": 2e-3}


# ---- the same in 64 bits ----------------------------------------------------------------


def _initial_h(seed, n, k):
    """The initial H that a handle's seed stands for: 0.1 z, z from the Box-Muller
    transform of two splitmix64 draws per entry."""
    def mix(x):
        x = x + np.uint64(0x9E3779B97F4A7C15)
        x = (x ^ (x >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        x = (x ^ (x >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return x ^ (x >> np.uint64(31))

    with np.errstate(over="ignore"):
        key = mix(np.array([seed], dtype=np.uint64))
        e = np.uint64(2) * np.arange(n * k, dtype=np.uint64)
        u1, u2 = ((mix(key + e + np.uint64(d)) >> np.uint64(11)).astype(np.float64) * 2.0 ** -53 for d in (0, 1))
    z = np.sqrt(-2.0 * np.log1p(-u1)) * np.cos(2.0 * np.pi * u2)
    return (0.1 * z).astype(np.float32).reshape(n, k)


class _Side:
    """Sums over the ratings of each row (or column): products with a sparse matrix."""

    def __init__(self, own, other, shape, order):
        self.order, self.shape = order, shape
        own, self.other = (own, other) if order is None else (own[order], other[order])
        count = torch.bincount(own.long(), minlength=shape[0])
        self.start = torch.cat([count.new_zeros(1), count.cumsum(0)]).to(torch.int32)
        self.ones = torch.ones(own.numel(), dtype=torch.float64, device="cuda")

    def sums(self, values, x):
        return (torch.sparse_csr_tensor(self.start, self.other, values, self.shape) @ x[:, None])[:, 0]

    def coordinate(self, rhat, x, lam):
        values = rhat if self.order is None else rhat[self.order]
        num, den = self.sums(values, x), lam + self.sums(self.ones, x * x)
        return torch.where(den == 0.0, torch.zeros_like(num), num / torch.where(den == 0.0, torch.ones_like(den), den))


def _predict(w, h, row, col):
    out = torch.zeros(row.numel(), dtype=torch.float64, device="cuda")
    for t in range(w.shape[1]):
        out += w[:, t][row] * h[:, t][col]
    return out


def exact(case, seed):
    train, held = _triplets(case, seed)
    w, h = _factors(case, seed)
    m, n, k, lam = case["m"], case["n"], case["k"], case["lam"]
    if case["kind"] == "fit":
        h = torch.from_numpy(_initial_h(int(seed) % (1 << 62), n, k)).cuda()
    w = torch.zeros(m, k, dtype=torch.float64, device="cuda") if w is None else w.double()
    h = h.double()

    def rmse(part):
        return float((part[2].double() - _predict(w, h, part[0], part[1])).square().mean().sqrt())

    if case["kind"] == "evaluate":
        return rmse(held)
    if case["nnz"] > 150_000_000:
        return None  # the sorted copies and the sums in 64 bits take too long
    row, col, val = train
    by_item = torch.argsort(col.long() * m + row.long())
    sides = (_Side(row, col, (m, n), None), _Side(col, row, (n, m), by_item))
    r = val.double() - _predict(w, h, row, col)
    history = []
    for _ in range(case["outer"]):
        if case["kind"] == "ccd":
            for s, (own, other) in enumerate(((w, h), (h, w))):
                for t in range(k):
                    r += w[:, t][row] * h[:, t][col]
                    own[:, t] = sides[s].coordinate(r, other[:, t].contiguous(), lam)
                    r -= w[:, t][row] * h[:, t][col]
            continue
        for t in range(k):
            u, v = w[:, t].contiguous(), h[:, t].contiguous()
            r += u[row] * v[col]
            for _ in range(case["inner"]):
                u = sides[0].coordinate(r, v, lam)
                v = sides[1].coordinate(r, u, lam)
            r -= u[row] * v[col]
            w[:, t], h[:, t] = u, v
        if case["kind"] == "monitor":
            sse = float(r.square().sum())
            f = sse + lam * float(w.square().sum() + h.square().sum())
            history.append([f, math.sqrt(sse / case["nnz"]), rmse(held)])
    out = (_host(w), _host(h))
    return (np.array(history),) + out if case["kind"] == "monitor" else out
