"""Workloads of the ROBE lookup path, for timing it and for comparing its results.

A case is one pass of a program that uses the library: a lookup (serving), a lookup with its
backward, or a whole training step, on inputs that are already on the GPU.  Sizes are those of the
repository's own configurations (1 GB and 100 MB arrays, 26 tables, d = 128) and of smaller and odd
ones of the same kinds.  Token ids follow the bounded Zipf law of click logs (exponent 1.05) over
table sizes spaced evenly on a log scale, or are uniform; bags have Poisson sizes, empty ones among them.

Fields of a case
  kind      "forward"    robe_forward (or _bf16, or _mixed)
            "step"       the gradient cleared, forward, backward
            "sgd"        forward, backward, robe_sgd_update: three calls
            "adagrad"    forward, robe_backward_adagrad
            "sgd_fused"  forward, robe_backward_sgd
  m, d, Z, sign          the ROBE instance
  tables, batch          lookups are [batch][tables]
  lo, hi                 table sizes, log-spaced from lo to hi
  alpha                  Zipf exponent of the ids, 0: uniform
  bag                    mean bag size, 0: single-hot
  mixed                  tables of 16 / 32 / 64 / 128 floats instead of d (the four quarters)
  bf16                   the array is a bfloat16 copy (forward only)
  repeatable             the reproducible option of the backward
"""
import math

import numpy as np
import torch

import paper_2108_02191_amd as robe

P = 2**31 - 1
SEED = 2108_02191
LR, EPS = 0.01, 1e-8
DEVICE = "cuda"


def _case(kind, m, d, Z, batch, **other):
    c = {"kind": kind, "m": m, "d": d, "Z": Z, "batch": batch, "tables": 26, "lo": 10, "hi": 40_000_000, "alpha": 1.05,
         "sign": 0, "bag": 0.0, "mixed": False, "bf16": False, "repeatable": False}
    c.update(other)
    return c


def listed():
    cases = {
        # a unit-sized model (4 MB array): what a first experiment or a test suite runs; launches count
        "tiny_step": _case("step", 2**20, 16, 4, 256, lo=1000, hi=1000, alpha=0.0),
        # a Kaggle-sized model (2 MB array, d = 16) trained with SGD as three calls
        "kaggle_sgd": _case("sgd", 540_000, 16, 4, 2048, lo=3, hi=10_131_227),
        # online serving: a few dozen requests per call, where latency is what counts
        "serve_64": _case("forward", 25_000_000, 128, 32, 64, sign=1),
        # batch inference on the 100 MB array
        "inference": _case("forward", 25_000_000, 128, 32, 32768, sign=1),
        # inference over bags on a quantised copy of the large array
        "bags_bf16": _case("forward", 250_000_000, 128, 32, 16384, lo=40_000_000, bag=20.0, bf16=True),
        # the training step of the 100 MB array
        "train_adagrad": _case("adagrad", 25_000_000, 128, 32, 65536),
        # per-element hashing, the far end of the block-size range
        "sweep_z1": _case("step", 25_000_000, 128, 1, 32768),
        # small blocks, in a run that has to give the same bits every time
        "repeatable_z8": _case("step", 25_000_000, 128, 8, 32768, repeatable=True),
        # tables of several dimensions in one array
        "mixed_step": _case("step", 25_000_000, 128, 16, 32768, mixed=True),
        # odd sizes throughout: d not a power of two, short bags, a ragged array and batch, signs
        "ragged_sgd": _case("sgd_fused", 6_000_011, 100, 10, 3001, tables=13, hi=1_000_003, sign=1, bag=3.0),
        # the 1 GB array with a small batch: frequent updates, most of the array untouched
        "large_array_256": _case("adagrad", 250_000_000, 128, 32, 256, lo=40_000_000, bag=20.0),
        # the 1 GB array with a full batch of bags
        "multihot": _case("adagrad", 250_000_000, 128, 32, 16384, lo=40_000_000, bag=20.0),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _block(rng, d, most=128):
    """A block size for dimension d: a divisor of it."""
    return rng.choice([z for z in (1, 2, 4, 5, 8, 10, 16, 25, 32, 64, 128) if d % z == 0 and z <= most])


def draw(rng):
    family = rng.choice(("small", "small", "serve", "serve", "inference", "bags", "train", "train", "sweep", "repeatable",
                         "mixed", "ragged", "large", "large"))
    big = lambda: _log(rng, 100_000, 40_000_000)  # noqa: E731
    if family == "small":
        d = rng.choice((8, 16, 24, 32))
        return _case(rng.choice(("step", "sgd")), _log(rng, 2**18, 2**22), d, _block(rng, d), _log(rng, 100, 6000),
                     tables=rng.randint(5, 40), lo=3, hi=big(), alpha=rng.choice((0.0, 1.05)))
    if family == "serve":
        d = rng.choice((16, 32, 64, 100, 128))
        return _case("forward", _log(rng, 5_000_000, 50_000_000), d, rng.choice((_block(rng, d), 4 * d)), _log(rng, 1, 2048),
                     tables=rng.randint(8, 40), hi=big(), sign=rng.randint(0, 1), bf16=rng.random() < 0.3)
    if family == "inference":
        d = rng.choice((64, 96, 128))
        return _case("forward", _log(rng, 10_000_000, 60_000_000), d, rng.choice((8, 16, 32)), _log(rng, 4096, 40000),
                     hi=big(), sign=rng.randint(0, 1), bf16=rng.random() < 0.3)
    if family == "bags":
        return _case("forward", _log(rng, 25_000_000, 250_000_000), rng.choice((64, 128)), rng.choice((16, 32, 64)), _log(rng, 1000, 16000),
                     hi=big(), bag=rng.uniform(2.0, 20.0), sign=rng.randint(0, 1), bf16=rng.random() < 0.5)
    if family == "train":
        d = rng.choice((64, 128))
        return _case(rng.choice(("adagrad", "adagrad", "sgd_fused")), _log(rng, 10_000_000, 60_000_000), d, rng.choice((8, 16, 32, 64)),
                     _log(rng, 8000, 66000), hi=big())
    if family == "sweep":
        return _case("step", _log(rng, 10_000_000, 50_000_000), 128, rng.choice((1, 2, 4, 8, 16, 32, 64, 128, 512)), _log(rng, 8000, 33000),
                     hi=big())
    if family == "repeatable":
        return _case(rng.choice(("step", "adagrad")), _log(rng, 10_000_000, 50_000_000), rng.choice((64, 128)), rng.choice((8, 16, 32)),
                     _log(rng, 2000, 33000), hi=big(), repeatable=True)
    if family == "mixed":
        return _case("step", _log(rng, 10_000_000, 50_000_000), 128, rng.choice((8, 16)), _log(rng, 1000, 33000),
                     tables=rng.randint(8, 32), hi=big(), mixed=True)
    if family == "ragged":
        d = rng.choice((20, 48, 100, 200))
        return _case(rng.choice(("step", "sgd_fused", "adagrad")), _log(rng, 1_000_000, 20_000_000), d, _block(rng, d), _log(rng, 500, 8000),
                     tables=rng.randint(5, 30), hi=big(), sign=rng.randint(0, 1), bag=rng.choice((0.0, rng.uniform(1.0, 6.0))))
    return _case(rng.choice(("adagrad", "adagrad", "sgd_fused")), _log(rng, 2**26, 250_000_000), 128, rng.choice((16, 32, 64)),
                 _log(rng, 50, 15000), lo=1_000_000, bag=rng.uniform(5.0, 20.0))


# ---------------------------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------------------------
def _cards(c):
    F = c["tables"]
    return [int(round(c["lo"] * (c["hi"] / c["lo"]) ** (f / max(1, F - 1)))) for f in range(F)]


def _dims(c):
    F = c["tables"]
    return [16 << (4 * f // F) for f in range(F)] if c["mixed"] else [c["d"]] * F


def _floats(c):
    """Floats of a sample's output row."""
    return sum(_dims(c))


HEAD = 4096     # ranks of a table whose probabilities are summed one by one; the rest by the integral of r^-alpha


def _zipf(c, u, table):
    """Ids from the bounded Zipf law by its inverse distribution function, u uniform in [0, 1)."""
    a = c["alpha"]
    head = np.cumsum(np.arange(1, HEAD + 1, dtype=np.float64) ** -a)
    first = (HEAD + 0.5) ** (1 - a)
    total = [head[n - 1] if n <= HEAD else head[-1] + (first - (n + 0.5) ** (1 - a)) / (a - 1) for n in _cards(c)]
    v = u * torch.tensor(total, dtype=torch.float64, device=DEVICE)[table]
    ids = torch.searchsorted(torch.from_numpy(head).to(DEVICE), v, right=True)
    tail = (first - (v - head[-1]).clamp_min(0.0) * (a - 1)) ** (1 / (1 - a))
    return torch.where(ids < HEAD, ids, (tail - 0.5).long().clamp_min(HEAD))


def _inputs(c, seed):
    """What a program has on the GPU before the call, from the seed alone (no arithmetic of the method)."""
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    F, B, m = c["tables"], c["batch"], c["m"]
    rows = B * F
    s = {"array": torch.randn(m, generator=gen, device=DEVICE).mul_(0.01)}
    offsets = None
    if c["bag"]:
        sizes = torch.poisson(torch.full((rows,), float(c["bag"]), device=DEVICE), generator=gen).long()
        offsets = torch.zeros(rows + 1, dtype=torch.int64, device=DEVICE)
        offsets[1:] = sizes.cumsum(0)
        row = torch.repeat_interleave(torch.arange(rows, device=DEVICE), sizes)
    else:
        row = torch.arange(rows, device=DEVICE)
    table = row % F
    cards = torch.tensor(_cards(c), dtype=torch.int64, device=DEVICE)[table]
    u = torch.rand(row.numel(), generator=gen, dtype=torch.float64, device=DEVICE)
    if c["alpha"]:
        ids = _zipf(c, u, table)
    else:
        ids = (u * cards).long()
    ids = torch.minimum(ids, cards - 1)
    s.update(indices=ids if c["bag"] else ids.view(B, F), offsets=offsets, row=row)
    if c["kind"] != "forward":
        s["grad_out"] = torch.randn(B, _floats(c), generator=gen, device=DEVICE)
    if c["kind"] in ("step", "sgd"):
        s["grad"] = torch.zeros(m, device=DEVICE)
    if c["kind"] == "sgd":                      # the gradient of a mean over the batch
        s["grad_out"] /= B
    if c["kind"] == "adagrad":                  # an accumulator some way into the training
        s["state"] = torch.rand(m, generator=gen, device=DEVICE).add_(0.5)
    return s


def prepare(case, seed):
    c = case
    s = _inputs(c, seed)
    del s["row"]
    s["c"] = {k: c[k] for k in ("kind", "batch", "tables", "mixed", "bf16")}
    h = s["hash"] = robe.robe_init_hash(SEED, c["m"], c["d"], c["Z"], c["sign"])
    s["dims"] = _dims(c)
    s["options"] = robe.options(reproducible=1) if c["repeatable"] else None
    if c["bf16"]:
        s["array"] = robe.robe_array_to_bf16(s["array"])
    n, B, F = s["indices"].numel(), c["batch"], c["tables"]
    if c["kind"] == "forward":
        need = 0
    elif c["kind"] in ("adagrad", "sgd_fused"):
        need = robe.robe_fused_workspace_bytes(h, B, F, n, s["options"])
    elif c["mixed"]:
        need = robe.robe_mixed_workspace_bytes(h, s["dims"], B, n, s["options"])
    else:
        need = robe.robe_workspace_bytes(h, B, F, n, s["options"])
    s["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEVICE) if need else None
    return s


def run(s):
    c, h, ids, offsets, opt, ws = s["c"], s["hash"], s["indices"], s["offsets"], s["options"], s["workspace"]
    kind, B, F, array = c["kind"], c["batch"], c["tables"], s["array"]
    if c["mixed"]:
        out = robe.robe_forward_mixed(h, s["dims"], array, ids, offsets, B)
    elif c["bf16"]:
        out = robe.robe_forward_bf16(h, array, ids, offsets, B, F)
    else:
        out = robe.robe_forward(h, array, ids, offsets, B, F)
    if kind == "forward":
        return [out]
    if kind == "adagrad":
        robe.robe_backward_adagrad(h, s["grad_out"], ids, offsets, B, F, array, s["state"], LR, EPS, workspace=ws, options=opt)
        return [out, array, s["state"]]
    if kind == "sgd_fused":
        robe.robe_backward_sgd(h, s["grad_out"], ids, offsets, B, F, array, LR, workspace=ws, options=opt)
        return [out, array]
    grad = s["grad"]
    if kind == "sgd":
        robe.robe_backward(h, s["grad_out"], ids, offsets, B, F, grad, workspace=ws, options=opt)
        robe.robe_sgd_update(h, array, grad, 1.0)
        return [out, array]
    grad.zero_()
    if c["mixed"]:
        robe.robe_backward_mixed(h, s["dims"], s["grad_out"], ids, offsets, B, grad, workspace=ws, options=opt)
    else:
        robe.robe_backward(h, s["grad_out"], ids, offsets, B, F, grad, workspace=ws, options=opt)
    return [out, grad]


# ---------------------------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------------------------
def _distinct(card, n, alpha):
    """Expected number of distinct ids among n draws from a table of `card` ids."""
    if not alpha:
        return card * -math.expm1(n * math.log1p(-1.0 / card)) if card > 1 else 1.0
    edge = np.unique(np.round(np.geomspace(1, card + 1, 400)).astype(np.int64)).astype(np.float64)
    lo, hi = edge[:-1], edge[1:]
    mass = np.where(hi - lo > 1, ((lo - 0.5) ** (1 - alpha) - (hi - 0.5) ** (1 - alpha)) / (alpha - 1), lo ** -alpha)
    p = mass / mass.sum() / (hi - lo)
    return float(((hi - lo) * -np.expm1(-n * p)).sum())


def work(case):
    c = case
    F, B, m = c["tables"], c["batch"], c["m"]
    dims, cards = _dims(c), _cards(c)
    per_table = B * (c["bag"] or 1.0)
    tokens = per_table * F
    reached = sum(_distinct(n, per_table, c["alpha"]) * d for n, d in zip(cards, dims))
    touched = m * -math.expm1(-reached / m)                     # slots that some token reads or writes
    rows = 4.0 * B * _floats(c)
    bags = 8.0 * (B * F + 1) if c["bag"] else 0.0
    moved = 8.0 * tokens + bags + (2 if c["bf16"] else 4) * touched + rows
    sums = per_table * sum(dims)
    if c["kind"] == "forward":
        return {"bytes": moved, "flops": sums}
    moved += rows                                               # the gradient rows
    rule = {"step": 4.0 * m, "sgd": 4.0 * touched, "sgd_fused": 4.0 * touched, "adagrad": 12.0 * touched}[c["kind"]]
    return {"bytes": moved + rule, "flops": 2 * sums + 6 * touched}


# Measured: 32-bit sums of bags and gradients are up to 1e-6 off exact() (frequent tokens have the
# longest sums), single values up to 7e-5 between two runs; values that are only moved are the same bits.
def tolerance(case):
    if case["kind"] == "forward" and not case["bag"]:
        return "exact"
    return {"rel": 4e-6, "max": 3e-4}


# ---------------------------------------------------------------------------------------------
# The same in 64 bits (Eq. 4 and 5 of the paper for the places, Eq. 2 for the signs)
# ---------------------------------------------------------------------------------------------
def _coefficients():
    """SplitMix64 from the seed, in the documented order A B C D of h, then of g."""
    state, got = SEED, []
    for k in range(8):
        state = (state + 0x9E3779B97F4A7C15) % 2**64
        z = state
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9 % 2**64
        z = (z ^ (z >> 27)) * 0x94D049BB133111EB % 2**64
        z ^= z >> 31
        got.append(z % P if k in (3, 7) else 1 + z % (P - 1))
    return got


def _places(c, x, e, d):
    """Array places and signs, [n][d], of the tokens x of the tables e."""
    A, B, C, D, Ag, Bg, Cg, Dg = _coefficients()
    Z, m = c["Z"], c["m"]
    i = torch.arange(d, device=x.device)
    chunk, inside, key = i // Z, i % Z, x
    if Z > d:                                   # Z / d consecutive tokens share a block
        r = Z // d
        key = x // r
        inside = (x % r)[:, None] * d + i
    start = ((A * e + B * key + D) % P)[:, None] + (C * chunk) % P
    place = (start % P % m + inside) % m
    if not c["sign"]:
        return place, None
    g = ((Ag * e + Bg * x + Dg) % P)[:, None] + (Cg * i) % P
    return place, (2 * (g % P % 2) - 1).double()


def exact(case, seed):
    c = case
    s = _inputs(c, seed)
    F, B = c["tables"], c["batch"]
    x, row, array = s["indices"].reshape(-1), s["row"], s["array"]
    source = array.to(torch.bfloat16) if c["bf16"] else array
    train = c["kind"] != "forward"
    out = torch.zeros(B, _floats(c), dtype=torch.float64, device=DEVICE)
    grad = torch.zeros(c["m"], dtype=torch.float64, device=DEVICE) if train else None
    # all tables at once, or (several dimensions) table by table; column: the tables' place in a sample's row
    views, column = [], 0
    for f, d in enumerate(_dims(c)):
        if not c["mixed"]:
            views = [(x, row, row % F, d, out.view(B * F, d), s["grad_out"].view(B * F, d) if train else None)]
            break
        mine = row % F == f
        views.append((x[mine], row[mine] // F, row[mine] % F, d, out[:, column:column + d], s["grad_out"][:, column:column + d] if train else None))
        column += d
    for vx, vrow, ve, d, vout, vgrad in views:
        step = max(1, 2**26 // d)
        for k in range(0, vx.numel(), step):
            to = vrow[k:k + step]
            place, sign = _places(c, vx[k:k + step], ve[k:k + step], d)
            v = source[place].double()
            vout.index_add_(0, to, v if sign is None else v * sign)
            if train:
                v = vgrad[to].double()
                grad.index_add_(0, place.reshape(-1), (v if sign is None else v * sign).reshape(-1))
    out = out if c["mixed"] else out.view(B, F, -1)
    if c["kind"] == "forward":
        return [out]
    if c["kind"] == "step":
        return [out, grad]
    if c["kind"] == "adagrad":
        state = s["state"].double() + grad * grad
        return [out, array.double() - float(np.float32(LR)) * grad / (state.sqrt() + float(np.float32(EPS))), state]
    return [out, array.double() - (1.0 if c["kind"] == "sgd" else float(np.float32(LR))) * grad]
