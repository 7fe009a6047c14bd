"""Performance cases of the FMM interaction library: the calls that a gravity
solver on 8^3 sub-grids makes, from one halo block to a 256^3-cell training
step, on seeded binary-star fields made on the GPU.

A case is a dict of plain values; its "kind" says which calls a pass makes:

  block   one 24^3 halo block (mono: the monopole form; jitter: how far the
          centres stray from a regular lattice)
  blocks  n halo blocks as event-polled futures of an Executor
  forward one batched forward (full: the full truncation; noalloc: the
          descriptor in device arrays instead of a plan)
  step    forward and gradients through autograd (save: the two-launch step,
          else the three-launch one)
  levels  a two-level gravity step: upward pass, fine forward and coarse
          substitutes, parent forward, downward pass, force and energy (amc:
          the fine forward with the angular-momentum correction)
  tree    the three tree passes alone

Batched cases work on a lattice of nx x ny x nz sub-grids, periodic or open;
a fraction `missing` of the targets lacks 1 to 9 of its 26 neighbours.
"""
import functools
import itertools
import math

import numpy as np
import torch

import paper_2303_08058_amd as ot

CELLS = 512
HALO3 = 24 ** 3
EXPS = [(a, b, n - a - b) for n in range(8) for a in range(n, -1, -1) for b in range(n - a, -1, -1)]
EXPS20 = EXPS[:20]
INV_FACT = [1.0 / (math.factorial(a) * math.factorial(b) * math.factorial(c)) for a, b, c in EXPS20]


def listed():
    return [
        # the monopole kernel on one halo block: the smallest call (leaf cells without moments)
        {"name": "block_monopole", "kind": "block", "mono": True, "jitter": 0.2},
        # the multipole kernel on one halo block: one sub-grid's call of a task-based solver
        {"name": "block_multipole", "kind": "block", "mono": False, "jitter": 0.2},
        # per-sub-grid launches as futures: the task-based solver itself, 64 sub-grids in flight
        {"name": "blocks_async", "kind": "blocks", "n": 64, "streams": 16, "workers": 2},
        # a coarse tree level: 27 sub-grids, open domain
        {"name": "forward_small", "kind": "forward", "nx": 3, "ny": 3, "nz": 3, "periodic": False,
         "missing": 0.0, "full": False, "noalloc": False},
        # a serving loop without plans: an odd box of sub-grids, tables in device arrays
        {"name": "forward_noalloc", "kind": "forward", "nx": 7, "ny": 6, "nz": 5, "periodic": True,
         "missing": 0.2, "full": False, "noalloc": True},
        # the batched forward of a 128^3-cell level
        {"name": "forward_4096", "kind": "forward", "nx": 16, "ny": 16, "nz": 16, "periodic": True,
         "missing": 0.15, "full": False, "noalloc": False},
        # forward and gradients of an isolated 64^3-cell system
        {"name": "step_open_512", "kind": "step", "nx": 8, "ny": 8, "nz": 8, "periodic": False,
         "missing": 0.0, "full": False, "save": True},
        # the step without saved sums (less memory), an odd box
        {"name": "step_two_pass_693", "kind": "step", "nx": 11, "ny": 9, "nz": 7, "periodic": True,
         "missing": 0.2, "full": False, "save": False},
        # the headline workload: forward and gradients of 256^3 cells
        {"name": "step_32768", "kind": "step", "nx": 32, "ny": 32, "nz": 32, "periodic": True,
         "missing": 0.2, "full": False, "save": True},
        # the same step under the full truncation, an odd box
        {"name": "full_step_720", "kind": "step", "nx": 10, "ny": 9, "nz": 8, "periodic": True,
         "missing": 0.2, "full": True, "save": True},
        # a whole gravity step over two levels, angular momentum conserved
        {"name": "levels_4096", "kind": "levels", "nx": 16, "ny": 16, "nz": 16, "periodic": True,
         "missing": 0.2, "full": False, "amc": True},
        # the memory-bound passes of a 256^3-cell level
        {"name": "tree_32768", "kind": "tree", "nx": 32, "ny": 32, "nz": 32},
    ]


def draw(rng):
    kind = rng.choice(["block", "blocks", "forward", "forward", "step", "step", "levels", "tree"])
    if kind == "block":
        return {"kind": kind, "mono": rng.random() < 0.5, "jitter": round(rng.uniform(0.05, 0.3), 3)}
    if kind == "blocks":
        return {"kind": kind, "n": int(2 ** rng.uniform(0, 8)), "streams": rng.randint(1, 32), "workers": rng.randint(0, 4)}
    full = rng.random() < 0.4
    # targets, log-uniform; the full truncation costs up to three times the total order a pair
    most = {"forward": 12 if full else 14, "step": 11 if full else 13, "levels": 12, "tree": 15}[kind]
    side = 2.0 ** (rng.uniform(0, most) / 3)
    n = [max(1, round(side * 2.0 ** rng.uniform(-0.4, 0.4))) for _ in range(3)]
    case = {"kind": kind}
    if kind in ("levels", "tree"):
        n = [2 * max(1, k // 2) for k in n]
    case.update(nx=n[0], ny=n[1], nz=n[2])
    if kind == "tree":
        return case
    # a periodic box of under 3 sub-grids would name a neighbour twice
    case["periodic"] = min(n) >= 3 and (kind != "levels" or min(n) >= 6) and rng.random() < 0.6
    case["missing"] = rng.choice([0.0, 0.15, 0.2, 0.5])
    case["full"] = full
    if kind == "forward":
        case["noalloc"] = not full and rng.random() < 0.3
    elif kind == "step":
        case["save"] = rng.random() < 0.7
    else:
        case["amc"] = not full and rng.random() < 0.5
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _moments(corner, dims, gen, sigmas, q, jitter=0.2):
    """Raw moments (20, n) about the centre of mass and centres (3, n) of the
    unit cells at integer `corner` (3, n) of a box of `dims` cells: 8 children
    a cell, jittered, sampling two Gaussian blobs over a floor density."""
    dev, n = corner.device, corner.shape[1]
    octant = torch.tensor([[i & 1, i >> 1 & 1, i >> 2] for i in range(8)], dtype=torch.float64, device=dev).T - 0.5
    x = corner[:, None, :] + 0.5 + 0.5 * octant[:, :, None]
    x = x + jitter * (torch.rand((3, 8, n), generator=gen, dtype=torch.float64, device=dev) - 0.5)
    rho = torch.full((8, n), 1e-10, dtype=torch.float64, device=dev)
    for side, s, amp in ((-5.0, sigmas[0], 1.0), (5.0, sigmas[1], q * (sigmas[0] / sigmas[1]) ** 3)):
        d2 = (x[0] - dims[0] / 2 - side) ** 2 + (x[1] - dims[1] / 2) ** 2 + (x[2] - dims[2] / 2) ** 2
        rho += amp * torch.exp(-d2 / (2 * s * s))
    m = rho * 0.125
    com = (m * x).sum(1) / m.sum(0)
    d = x - com[:, None, :]
    M = torch.stack([(m * d[0] ** a * d[1] ** b * d[2] ** c).sum(0) for a, b, c in EXPS20])
    return M, com


def _generator(seed):
    gen = torch.Generator(device=_device())
    gen.manual_seed(int(seed))
    return gen


def _block(seed, mono, jitter=0.2):
    gen, dev = _generator(seed), _device()
    i = torch.arange(HALO3, device=dev)
    corner = torch.stack([i % 24, i // 24 % 24, i // 576]).double()
    if mono:
        stray = jitter * (torch.rand((3, HALO3), generator=gen, dtype=torch.float64, device=dev) - 0.5)
        return 0.5 + torch.rand(HALO3, generator=gen, dtype=torch.float64, device=dev), corner + 0.5 + stray
    return _moments(corner, (24, 24, 24), gen, (3.0, 3.0), 0.7, jitter)


def _dims(case):
    return case["nx"], case["ny"], case["nz"]


def _store(dims, seed):
    """Moments (20, S*512) and centres (3, S*512) of a lattice of sub-grids."""
    gen, dev, S = _generator(seed), _device(), dims[0] * dims[1] * dims[2]
    pick = np.random.default_rng(seed)
    sigmas, q = pick.choice([2.0, 4.0], 2), pick.uniform(0.3, 1.0)
    M = torch.empty((20, S * CELLS), dtype=torch.float64, device=dev)
    X = torch.empty((3, S * CELLS), dtype=torch.float64, device=dev)
    c = torch.arange(CELLS, device=dev)
    cell = torch.stack([c % 8, c // 8 % 8, c // 64])
    for s0 in range(0, S, 4096):
        s = torch.arange(s0, min(S, s0 + 4096), device=dev)
        sub = torch.stack([s % dims[0], s // dims[0] % dims[1], s // (dims[0] * dims[1])])
        corner = (8 * sub[:, :, None] + cell[:, None, :]).reshape(3, -1).double()
        at = slice(s0 * CELLS, s0 * CELLS + corner.shape[1])
        M[:, at], X[:, at] = _moments(corner, [8 * k for k in dims], gen, sigmas, q)
    return M, X


def _lattice(dims, periodic, missing=0.0, seed=0, cell=1.0):
    """Descriptor of a lattice, all sub-grids targets, seeded missing neighbours."""
    S = dims[0] * dims[1] * dims[2]
    s = np.arange(S)
    at = np.stack([s % dims[0], s // dims[0] % dims[1], s // (dims[0] * dims[1])], 1)
    off = np.array([(q % 3 - 1, q // 3 % 3 - 1, q // 9 - 1) for q in range(27)])
    to = at[:, None, :] + off[None]
    wrapped = np.mod(to, dims)
    whole = (wrapped[..., 0] + dims[0] * (wrapped[..., 1] + dims[1] * wrapped[..., 2])).astype(np.int32)
    b = {"S": S, "T": S, "tgt": s.astype(np.int32), "shift": None, "period": None}
    if periodic:
        b["shift"] = ((to - wrapped) // dims).astype(np.int8)
        b["period"] = 8.0 * cell * np.array(dims, np.float64)
    else:
        whole = np.where((to == wrapped).all(-1), whole, -1).astype(np.int32)
    nbr = whole.copy()
    rng = np.random.default_rng(seed)
    hit = rng.random(S) < missing
    rank = np.argsort(np.argsort(rng.random((S, 26)), 1), 1)
    drop = np.insert(rank < rng.integers(1, 10, S)[:, None], 13, False, axis=1) & hit[:, None]
    nbr[drop] = -1
    b["nbr"], b["whole"] = nbr, whole
    return b


def _children(dims):
    m = [k // 2 for k in dims]
    P, o = np.arange(m[0] * m[1] * m[2]), np.arange(8)
    p = np.stack([P % m[0], P // m[0] % m[1], P // (m[0] * m[1])], 1)
    c = 2 * p[:, None, :] + np.stack([o & 1, o >> 1 & 1, o >> 2], 1)[None]
    return (c[..., 0] + dims[0] * (c[..., 1] + dims[1] * c[..., 2])).astype(np.int32)


def _substitutes(dims, b):
    """(node, octant) of the parent level that covers each neighbour a target lacks."""
    lost = np.where((b["nbr"] < 0) & (b["whole"] >= 0), b["whole"], -1)
    x, y, z = lost % dims[0], lost // dims[0] % dims[1], lost // (dims[0] * dims[1])
    node = x // 2 + dims[0] // 2 * (y // 2 + dims[1] // 2 * (z // 2))
    octant = x % 2 + 2 * (y % 2) + 4 * (z % 2)
    return np.where(lost >= 0, node, -1).astype(np.int32), np.where(lost >= 0, octant, 0).astype(np.int8)


def _empty(*shape):
    return torch.empty(shape, dtype=torch.float64, device=_device())


def _plan(b):
    return ot.Plan(b["S"], b["T"], b["tgt"], b["nbr"], b["shift"], b["period"])


def prepare(case, seed):
    kind = case["kind"]
    if kind == "block":
        M, X = _block(seed, case["mono"], case["jitter"])
        return {"case": case, "M": M, "X": X, "L": _empty(20, CELLS)}
    if kind == "blocks":
        # a solver's sub-grids: every block its own jitter and moments
        return {"case": case, "in": [_block(1000 * seed + i, False) for i in range(case["n"])],
                "L": _empty(case["n"], 20, CELLS), "ex": ot.Executor(case["streams"], case["workers"])}
    dims = _dims(case)
    M, X = _store(dims, seed)
    s = {"case": case, "M": M, "X": X}
    if kind == "tree":
        s.update(tree=ot.Tree(_children(dims), M.shape[1] // CELLS), Mp=_empty(20, M.shape[1] // 8),
                 Xp=_empty(3, M.shape[1] // 8), F=_empty(3, M.shape[1]), W=_empty(M.shape[1]),
                 **_expansions(M.shape[1], seed))
        return s
    b = _lattice(dims, case["periodic"], case["missing"], seed)
    N = b["T"] * CELLS
    if kind == "forward":
        s["L"] = _empty(20, N)
        if case["noalloc"]:
            dev = _device()
            s["b"] = {k: (torch.from_numpy(v).to(dev) if isinstance(v, np.ndarray) and k != "period" else v)
                      for k, v in b.items()}
        else:
            s["plan"] = _plan(b)
    elif kind == "step":
        M.requires_grad_(True)
        X.requires_grad_(True)
        s.update(plan=_plan(b), gL=torch.randn((20, N), generator=_generator(seed + 1), dtype=torch.float64, device=_device()))
    else:
        children = _children(dims)
        Sp = len(children)
        s.update(tree=ot.Tree(children, b["S"]), plan=_plan(b),
                 parent=_plan(_lattice([k // 2 for k in dims], case["periodic"], cell=2.0)),
                 Mp=_empty(20, Sp * CELLS), Xp=_empty(3, Sp * CELLS), L=_empty(20, N), Lp=_empty(20, Sp * CELLS),
                 F=_empty(3, N), W=_empty(N), dF=_empty(3, N))
        node, octant = _substitutes(dims, b)
        s["coarse"] = bool((node >= 0).any())
        if s["coarse"]:
            s["plan"].set_coarse(Sp, node, octant)
    return s


def _expansions(n, seed):
    """Local coefficients of a level and of its parent level."""
    gen = _generator(seed + 2)
    scale = torch.tensor([0.5 ** sum(e) for e in EXPS20], dtype=torch.float64, device=_device())[:, None]
    return {"L": torch.randn((20, n), generator=gen, dtype=torch.float64, device=_device()),
            "Lp": scale * torch.randn((20, n // 8), generator=gen, dtype=torch.float64, device=_device())}


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(state):
    return _RUN[state["case"]["kind"]](state["case"], state)


def _run_block(case, s):
    return (ot.ot_fmm_monopole if case["mono"] else ot.ot_fmm_multipole)(s["M"], s["X"], s["L"])


def _run_blocks(case, s):
    futures = [s["ex"].multipole_async(M, X, L) for (M, X), L in zip(s["in"], s["L"])]
    for f in futures:
        f.wait()
    return s["L"]


def _run_forward(case, s):
    if case["noalloc"]:
        b = s["b"]
        return ot.ot_fmm_multipole_batched_noalloc(b["S"], b["T"], b["tgt"], b["nbr"], b["shift"], b["period"],
                                                   s["M"], s["X"], s["L"])
    return (s["plan"].multipole_batched_full if case["full"] else s["plan"].multipole_batched)(s["M"], s["X"], s["L"])


def _run_step(case, s):
    M, X = s["M"], s["X"]
    M.grad = X.grad = None
    L = ot.multipole(M, X, s["plan"], case["full"], case["save"])
    L.backward(s["gL"])
    return {"L": L.detach(), "gM": M.grad, "gX": X.grad}


def _run_levels(case, s):
    plan, parent, M, X, L = s["plan"], s["parent"], s["M"], s["X"], s["L"]
    s["tree"].m2m(M, X, s["Mp"], s["Xp"])
    if case["amc"]:
        plan.multipole_batched_amc(M, X, L, s["dF"])
    elif case["full"]:
        plan.multipole_batched_full(M, X, L)
    else:
        plan.multipole_batched(M, X, L)
    if s["coarse"]:
        plan.coarse_fine(X, s["Mp"], s["Xp"], L, full=case["full"])
    (parent.multipole_batched_full if case["full"] else parent.multipole_batched)(s["Mp"], s["Xp"], s["Lp"])
    s["tree"].l2l(s["Lp"], s["Xp"], X, L)
    ot.ot_fmm_evaluate(M, L, s["F"], s["W"])
    out = {"L": L, "F": s["F"], "W": s["W"]}
    if case["amc"]:
        out["F"] += s["dF"]
    return out


def _run_tree(case, s):
    # the downward pass adds into the coefficients it is given: a pass starts from the same ones
    s["tree"].m2m(s["M"], s["X"], s["Mp"], s["Xp"])
    L = s["L"].clone()
    s["tree"].l2l(s["Lp"], s["Xp"], s["X"], L)
    ot.ot_fmm_evaluate(s["M"], L, s["F"], s["W"])
    return {"Mp": s["Mp"], "Xp": s["Xp"], "L": L, "F": s["F"], "W": s["W"]}


_RUN = {"block": _run_block, "blocks": _run_blocks, "forward": _run_forward, "step": _run_step,
        "levels": _run_levels, "tree": _run_tree}


# ---------------------------------------------------------------------------
# bytes and operations
# ---------------------------------------------------------------------------
def _criterion(i, j):
    d = j - i
    p = j // 2 - i // 2
    return ((d * d).sum(-1) > 16) & ((p * p).sum(-1) <= 16)


@functools.lru_cache(None)
def _slot_pairs():
    c = np.arange(CELLS)
    local = np.stack([c % 8, c // 8 % 8, c // 64], 1)
    return [int(_criterion(8 + local[:, None], 8 * np.array([q % 3, q // 3 % 3, q // 9]) + local[None]).sum())
            for q in range(27)]


# FP64 operations of a pair, FMA = 2, with the contraction arranged around the
# separation vector: the forward's order-3 sums, the sums of total order 4 for
# one role, both sets, and the same under the full truncation
_FORWARD, _ROLE, _BOTH, _FULL, _FULL4 = 165, 275, 345, 340, 520


def work(case):
    kind = case["kind"]
    if kind in ("block", "blocks"):
        n, mono = case.get("n", 1), case.get("mono", False)
        return {"bytes": n * 8 * ((4 if mono else 23) * HALO3 + 20 * CELLS),
                "flops": n * sum(_slot_pairs()) * (90 if mono else _FORWARD)}
    dims = _dims(case)
    S = dims[0] * dims[1] * dims[2]
    N = S * CELLS
    tree = {"bytes": 8 * N * (23 + 23 / 8 + 23 / 8 + 3 + 40 + 40 + 4), "flops": N * (400 + 260 + 120)}
    if kind == "tree":
        return tree
    pairs = sum(n * math.prod(d if case["periodic"] else max(0, d - abs(o)) for d, o in
                              zip(dims, (q % 3 - 1, q // 3 % 3 - 1, q // 9 - 1)))
                * (1.0 if q == 13 else 1.0 - case["missing"] * 5 / 26) for q, n in enumerate(_slot_pairs()))
    full = case["full"]
    forward = {"bytes": 8 * N * 43, "flops": pairs * (_FULL if full else _FORWARD)}
    if kind == "forward":
        return forward
    if kind == "step":
        if case["save"]:
            return {"bytes": 8 * N * (23 + 20 + 24 + 43 + 24 + 23), "flops": pairs * 2 * (_FULL4 if full else _BOTH)}
        return {"bytes": 8 * N * (43 + 43 + 23), "flops": pairs * ((_FULL + 2 * _FULL4) if full else (_FORWARD + _BOTH + _ROLE))}
    both = forward["flops"] * (1 + 1 / 8) + (pairs * (_BOTH - _FORWARD) if case["amc"] else 0)
    return {"bytes": tree["bytes"] + 8 * N * (43 + 43 / 8 + (6 if case["amc"] else 0)), "flops": tree["flops"] + both}


# ---------------------------------------------------------------------------
# the same results in plain torch
# ---------------------------------------------------------------------------
def _derivatives(r, order):
    """G_g(r), G = -1/|r|, for every |g| <= order: chain rule on the radial factors."""
    r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2]
    D = [-1.0 / torch.sqrt(r2)]
    for p in range(order):
        D.append(D[-1] * (-(2 * p + 1)) / r2)

    @functools.lru_cache(None)
    def phi(p, e):
        if e == (0, 0, 0):
            return D[p]
        k = next(i for i in (2, 0, 1) if e[i] > 0)
        less = tuple(v - (i == k) for i, v in enumerate(e))
        out = r[k] * phi(p + 1, less)
        if less[k] > 0:
            out = torch.add(out, phi(p + 1, tuple(v - (i == k) for i, v in enumerate(less))), alpha=less[k])
        return out

    return {e: phi(0, e) for e in EXPS if sum(e) <= order}


def _terms(r, m, full, weight=None):
    """The 20 outputs of pairs with separations r (3, ...) and source moments m
    (20, ...); `weight`: the targets' moments over factorials, for the force correction."""
    G = _derivatives(r, 6 if full else (4 if weight is not None else 3))
    q = [(-1.0 if sum(b) % 2 else 1.0) * INV_FACT[i] * m[i] for i, b in enumerate(EXPS20)]
    out = []
    for a in EXPS20:
        v = torch.zeros_like(r[0])
        for i, b in enumerate(EXPS20):
            if full or sum(a) + sum(b) <= 3:
                v = torch.addcmul(v, q[i], G[tuple(x + y for x, y in zip(a, b))])
        out.append(v)
    if weight is not None:
        for k in range(3):
            v = torch.zeros_like(r[0])
            for (i, a), (j, b) in itertools.product(enumerate(EXPS20), repeat=2):
                if sum(a) + sum(b) == 3:
                    v = torch.addcmul(v, weight[i] * q[j], G[tuple(x + y + (n == k) for n, (x, y) in enumerate(zip(a, b)))], value=-1.0)
            out.append(v)
    return out


@functools.lru_cache(None)
def _offsets(parity):
    """The targets of one parity (64 cells) and, for each offset of its stencil, their sources' slots and cells."""
    o = np.stack(np.meshgrid(*[np.arange(-9, 10)] * 3, indexing="ij"), -1).reshape(-1, 3)
    base = 8 + np.array(parity)
    o = o[_criterion(base[None], base[None] + o)]
    c = np.arange(CELLS)
    local = np.stack([c % 8, c // 8 % 8, c // 64], 1)
    mine = local[(local % 2 == np.array(parity)).all(1)]
    h = 8 + mine[None] + o[:, None]
    slot = h[..., 0] // 8 + 3 * (h[..., 1] // 8) + 9 * (h[..., 2] // 8)
    cell = h[..., 0] % 8 + 8 * (h[..., 1] % 8) + 64 * (h[..., 2] % 8)
    return mine @ np.array([1, 8, 64]), slot, cell


def _interaction(M, X, b, full=False, amc=False, gL=None):
    """L (and the force correction, 23 rows, with amc) of a lattice descriptor;
    with gL the gradients are left in M.grad and X.grad."""
    dev, T = M.device, b["T"]
    nbr = torch.from_numpy(b["nbr"].astype(np.int64)).to(dev)
    shift = torch.zeros((T, 27, 3), dtype=torch.float64, device=dev)
    if b["shift"] is not None:
        shift = torch.from_numpy(b["shift"] * b["period"]).to(dev)
    L = torch.zeros((23 if amc else 20, T, CELLS), dtype=torch.float64, device=dev)
    fact = torch.tensor(INV_FACT, dtype=torch.float64, device=dev)[:, None]
    step = max(1, (1 << 22) // (64 * T))
    for parity in itertools.product((0, 1), repeat=3):
        mine, slot, cell = (torch.from_numpy(np.ascontiguousarray(v)).to(dev) for v in _offsets(parity))
        own = (CELLS * torch.arange(T, device=dev)[:, None] + mine[None]).reshape(-1)
        for k in range(0, slot.shape[0], step):
            sl, ce = slot[k:k + step], cell[k:k + step]
            block = nbr[:, sl].permute(1, 0, 2)                       # offsets, targets, cells
            there = block >= 0
            src = (block.clamp(min=0) * CELLS + ce[:, None, :]).reshape(-1)
            n = sl.shape[0]
            xi = X[:, own][:, None].expand(3, n, own.numel())
            xj = X[:, src].reshape(3, n, -1) + shift[:, sl].permute(3, 1, 0, 2).reshape(3, n, -1)
            m = M[:, src].reshape(20, n, -1) * there.reshape(n, -1)
            weight = (M[:, own] * fact)[:, None] if amc else None
            r = torch.where(there.reshape(n, -1), xi - xj, 1.0)
            out = torch.stack([v.sum(0) for v in _terms(r, m, full, weight)])
            if gL is not None:
                out.backward(gL.reshape(20, T, CELLS)[:, :, mine].reshape(20, -1))
            L[:, :, mine] += out.detach().reshape(-1, T, mine.numel())
    return L.reshape(L.shape[0], -1)


def _coarse(X, Mp, Xp, b, node, octant, full):
    """The coarse substitutes' part of L."""
    dev, T = X.device, b["T"]
    c, J = np.arange(CELLS), np.arange(64)
    hi = 8 + np.stack([c % 8, c // 8 % 8, c // 64], 1)
    cj = np.stack([J % 4, J // 4 % 4, J // 16], 1)
    L = torch.zeros((20, T * CELLS), dtype=torch.float64, device=dev)
    for q in range(27):
        t = np.nonzero(node[:, q] >= 0)[0]
        if not len(t):
            continue
        first = 8 * np.array([q % 3, q // 3 % 3, q // 9]) + 2 * cj
        inside = np.ones((CELLS, 64), bool)
        for o in itertools.product((0, 1), repeat=3):
            inside &= _criterion(hi[:, None], first[None] + np.array(o))
        pc, pJ = np.nonzero(inside)
        for part in np.array_split(t, max(1, len(t) * len(pc) // (1 << 22))):
            o = octant[part, q].astype(np.int64)[:, None]
            k = cj[pJ][None] + 4 * np.stack([o & 1, o >> 1 & 1, o >> 2], -1)
            src = torch.from_numpy((node[part, q].astype(np.int64)[:, None] * CELLS + k @ np.array([1, 8, 64])).reshape(-1)).to(dev)
            own = torch.from_numpy((part[:, None] * CELLS + pc[None]).reshape(-1)).to(dev)
            xj = Xp[:, src]
            if b["shift"] is not None:
                xj = xj + torch.from_numpy(np.repeat(b["shift"][part, q] * b["period"], len(pc), 0).T).to(dev)
            L.index_add_(1, own, torch.stack(_terms(X[:, own] - xj, Mp[:, src], full)))
    return L


def _power(d, e):
    return d[0] ** e[0] * d[1] ** e[1] * d[2] ** e[2]


@functools.lru_cache(None)
def _family(dims):
    """Child cells (8, parent cells) of each parent cell."""
    ch = _children(dims).astype(np.int64)
    c = np.arange(CELLS)
    p = np.stack([c % 8, c // 8 % 8, c // 64], 1)
    o = p // 4 @ np.array([1, 2, 4])
    kids = [ch[:, o] * CELLS + (2 * (p % 4) + np.array(k)) @ np.array([1, 8, 64]) for k in itertools.product((0, 1), repeat=3)]
    return torch.from_numpy(np.stack(kids).reshape(8, -1))


def _up(dims, M, X):
    kids = _family(dims).to(M.device)
    m, x = M[:, kids], X[:, kids]
    mass = m[0].sum(0)
    Xp = torch.where(mass > 0, (m[0] * x).sum(1) / mass, x.mean(1))
    d = x - Xp[:, None]
    Mp = torch.zeros((20, Xp.shape[1]), dtype=M.dtype, device=M.device)
    for i, b in enumerate(EXPS20):
        for j, g in enumerate(EXPS20):
            if all(v <= u for u, v in zip(b, g)):
                binom = math.prod(math.comb(u, v) for u, v in zip(b, g))
                Mp[i] += binom * (m[j] * _power(d, [u - v for u, v in zip(b, g)])).sum(0)
    return Mp, Xp


def _down(dims, Lp, Xp, X, L):
    kids = _family(dims).to(L.device)
    d = X[:, kids] - Xp[:, None]
    out = L.clone()
    for i, a in enumerate(EXPS20):
        for j, g in enumerate(EXPS20):
            if sum(a) + sum(g) <= 3:
                out[i, kids] += INV_FACT[j] * Lp[EXPS20.index(tuple(u + v for u, v in zip(a, g)))] * _power(d, g)
    return out


def _force(M, L):
    F, W = torch.zeros_like(L[:3]), torch.zeros_like(L[0])
    for i, a in enumerate(EXPS20):
        W += 0.5 * INV_FACT[i] * M[i] * L[i]
        if sum(a) <= 2:
            for k in range(3):
                F[k] -= INV_FACT[i] * M[i] * L[EXPS20.index(tuple(u + (n == k) for n, u in enumerate(a)))]
    return F, W


def _exact_block(M, X, mono):
    if mono:
        M = torch.cat([M[None], torch.zeros((19, HALO3), dtype=torch.float64, device=M.device)])
    # the halo block as a store of 27 sub-grids with one target
    i = torch.arange(27 * CELLS, device=M.device)
    s, c = i // CELLS, i % CELLS
    h = (8 * (s % 3) + c % 8) + 24 * (8 * (s // 3 % 3) + c // 8 % 8) + 576 * (8 * (s // 9) + c // 64)
    order = torch.cat([torch.tensor([13]), torch.arange(13), torch.arange(14, 27)]).to(M.device)
    h = h.reshape(27, CELLS)[order].reshape(-1)
    nbr = np.argsort(order.cpu().numpy())[None]
    return _interaction(M[:, h], X[:, h], {"T": 1, "nbr": nbr, "shift": None})


def exact(case, seed):
    kind = case["kind"]
    if kind == "block":
        return _exact_block(*_block(seed, case["mono"], case["jitter"]), case["mono"])
    if kind == "blocks":
        return torch.stack([_exact_block(*_block(1000 * seed + i, False), False) for i in range(case["n"])]) if case["n"] <= 64 else None
    dims = _dims(case)
    T = dims[0] * dims[1] * dims[2]
    if kind == "tree":
        M, X = _store(dims, seed)
        e = _expansions(T * CELLS, seed)
        Mp, Xp = _up(dims, M, X)
        L = _down(dims, e["Lp"], Xp, X, e["L"])
        F, W = _force(M, L)
        return {"Mp": Mp, "Xp": Xp, "L": L, "F": F, "W": W}
    full = case["full"]
    if T > {"forward": 4096, "step": 1000, "levels": 4096}[kind] // (2 if full and kind != "step" else 1):
        return None
    M, X = _store(dims, seed)
    b = _lattice(dims, case["periodic"], case["missing"], seed)
    if kind == "forward":
        return _interaction(M, X, b, full)
    if kind == "step":
        M.requires_grad_(True)
        X.requires_grad_(True)
        gL = torch.randn((20, T * CELLS), generator=_generator(seed + 1), dtype=torch.float64, device=M.device)
        L = _interaction(M, X, b, full, gL=gL)
        return {"L": L, "gM": M.grad, "gX": X.grad}
    Mp, Xp = _up(dims, M, X)
    L = _interaction(M, X, b, full, amc=case["amc"])
    dF, L = L[20:], L[:20] + _coarse(X, Mp, Xp, b, *_substitutes(dims, b), full)
    Lp = _interaction(Mp, Xp, _lattice([k // 2 for k in dims], case["periodic"], cell=2.0), full)
    L = _down(dims, Lp, Xp, X, L)
    F, W = _force(M, L)
    return {"L": L, "F": F + dF if case["amc"] else F, "W": W}
