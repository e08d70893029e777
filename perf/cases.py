"""The work that users of this framework have it do, as cases that can be timed and compared.

A case is a plain dict. Two kinds of work:

``solve``   a solver with its game on the GPU runs ``iters`` CFR iterations and hands back the
            average strategy and, where the path has one (``check``), the exploitability of the
            average: the loop "iterate, look at the strategy, iterate on" that every solve is.
            ``game`` names the generator: Kuhn- and Leduc-shaped games, the multi-round poker game,
            a batch of poker subgames, a general-sum game of several players. The seed draws
            what differs from one solve to the next in use: the chance distribution at the root
            (the beliefs over private cards or types), the payoffs of a general-sum game, and the
            regrets that the solve is warm-started with (no iteration counted, no average yet).
            Tree shapes come from the case alone.
``net``     the warm-start network: prediction of strategies for a set of infosets (features from
            descriptors, forward pass, distribution over the legal actions), the forward pass
            alone, or training steps.

``exact`` computes the same in 64 bits with plain torch: level by level over a breadth-first
order of the game that it derives itself from the game's own arrays.
"""
from __future__ import annotations

import dataclasses
import functools
import math

import numpy as np
import torch

import games
from games.tuple import Game
from paper_2408_14778_amd import BatchSolver, NPlayerSolver, PartitionedSolver, Solver
from paper_2408_14778_amd import warmstart

DEVICE = "cuda"


def listed():
    return [
        # the smallest call: the 55-node Kuhn-shaped game, vanilla CFR in a long run (latency
        # and launches are all there is)
        {"name": "kuhn_vanilla", "do": "solve", "game": "kuhn", "ranks": 3, "variant": "vanilla",
         "schedule": "simultaneous", "precision": "f32", "iters": 100, "check": False},
        # an ordinary small study: the 100,981-node Leduc-shaped game, CFR+, with the
        # exploitability looked at every ten iterations
        {"name": "leduc_plus_check", "do": "solve", "game": "leduc", "ranks": 6, "suits": 2,
         "variant": "cfr+", "schedule": "simultaneous", "precision": "f32", "iters": 10,
         "check": True},
        # the large single game (21.5M nodes), CFR+: the framework's headline workload
        {"name": "poker_large_plus", "do": "solve", "game": "poker", "ranks": 13, "rounds": 3,
         "cap": 3, "stack": 400, "deals": 156, "variant": "cfr+", "schedule": "simultaneous",
         "precision": "f32", "iters": 10, "check": False},
        # a middle-sized odd one (a third of the deals of a 12-rank game), discounted CFR with
        # alternating updates
        {"name": "poker_mid_dcfr_alternating", "do": "solve", "game": "poker", "ranks": 12,
         "rounds": 3, "cap": 2, "stack": 300, "deals": 43, "variant": "dcfr",
         "schedule": "alternating", "precision": "f32", "iters": 10, "check": True},
        # double precision on a middle-sized game (the first 16 deals of the large one: the
        # sample that the CPU baseline takes), CFR+ with its exploitability
        {"name": "poker_mid_f64", "do": "solve", "game": "poker", "ranks": 13, "rounds": 3,
         "cap": 3, "stack": 400, "deals": 16, "variant": "cfr+", "schedule": "simultaneous",
         "precision": "f64", "iters": 10, "check": True},
        # many subgames at once: 48 poker subgames of mixed sizes, CFR+, every subgame's
        # exploitability every ten iterations (the batched solve loop)
        {"name": "subgames_48", "do": "solve", "game": "batch", "first": 100, "count": 48,
         "variant": "cfr+", "schedule": "simultaneous", "precision": "f32", "iters": 10,
         "check": True},
        # a three-player general-sum game of about two million nodes, CFR+
        {"name": "three_player", "do": "solve", "game": "public_n", "players": 3, "types": 12,
         "depth": 9, "tree": 1231, "variant": "cfr+", "schedule": "simultaneous",
         "precision": "f32", "iters": 10, "check": False},
        # a small general-sum game in double precision, a pass per player (three-player Kuhn)
        {"name": "kuhn3_f64_alternating", "do": "solve", "game": "kuhn3", "ranks": 4,
         "variant": "cfr+", "schedule": "alternating", "precision": "f64", "iters": 20,
         "check": False},
        # out of core: a poker game streamed through a window of 2^18 nodes
        {"name": "poker_out_of_core", "do": "solve", "game": "poker", "ranks": 13, "rounds": 3,
         "cap": 3, "stack": 400, "deals": 24, "variant": "cfr+", "schedule": "simultaneous",
         "precision": "f32", "iters": 4, "check": False, "cut": 7, "window": 1 << 18},
        # strategies of a batch's infosets from the network: features, forward, distributions
        {"name": "net_predict", "do": "net", "what": "predict", "rows": 200001, "hidden": 256},
        # the forward pass alone on one full batch
        {"name": "net_forward", "do": "net", "what": "forward", "rows": 65536, "hidden": 256},
        # training: mini-batches of 4,096 infosets, with the gradients and weights read back
        {"name": "net_train", "do": "net", "what": "train", "rows": 4096, "hidden": 256,
         "steps": 8},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["small", "leduc", "poker", "poker", "f64", "batch", "n", "n", "core",
                       "predict", "forward", "train"])
    variant = rng.choice(["vanilla", "cfr+", "dcfr"])
    schedule = rng.choice(["simultaneous", "simultaneous", "alternating"])
    base = {"do": "solve", "variant": variant, "schedule": schedule, "precision": "f32",
            "iters": rng.randint(6, 14), "check": rng.random() < 0.5}
    if what == "small":
        return {**base, "game": "kuhn", "ranks": rng.randint(3, 40), "iters": _log(rng, 20, 120),
                "precision": rng.choice(["f32", "f64"])}
    if what == "leduc":
        return {**base, "game": "leduc", "ranks": rng.randint(3, 6), "suits": 2,
                "precision": rng.choice(["f32", "f64"])}
    if what in ("poker", "f64", "core"):
        ranks, rounds, cap = rng.randint(7, 13), rng.randint(2, 3), rng.randint(1, 3)
        stack = rng.choice([20, 60, 150, 300, 400])
        per = games.template_size(ranks, rounds, cap, stack)
        deals = max(3, min(ranks * (ranks - 1), _log(rng, 2e4, 6e6) // per))
        case = {**base, "game": "poker", "ranks": ranks, "rounds": rounds, "cap": cap,
                "stack": stack, "deals": deals}
        if what == "f64":
            case["precision"] = "f64"
        if what == "core":
            case.update(cut=rng.randint(3, 5), window=_log(rng, 2e4, 5e5), check=False,
                        precision=rng.choice(["f32", "f32", "f64"]), iters=rng.randint(2, 6))
        return case
    if what == "batch":
        return {**base, "game": "batch", "first": rng.randint(100, 580),
                "count": rng.randint(3, 32), "check": True}
    if what == "n":
        players = rng.randint(3, 5)
        return {**base, "game": "public_n", "players": players,
                "types": rng.randint(2, {3: 12, 4: 6, 5: 4}[players]), "depth": rng.randint(5, 9),
                "tree": _log(rng, 60, 1500), "check": False,
                "precision": rng.choice(["f32", "f64"])}
    hidden = rng.choice([128, 256, 256])
    if what == "train":
        return {"do": "net", "what": "train", "rows": _log(rng, 300, 8000), "hidden": hidden,
                "steps": rng.randint(2, 10)}
    return {"do": "net", "what": what, "rows": _log(rng, 50, 200000), "hidden": hidden}


# ------------------------------------------------------------------------------ games


def _public_tree(depth: int, size: int):
    """A public tree of ``size`` nodes or a few fewer, of at most ``depth`` + 1 levels, grown
    breadth first (0: terminal, 1 ..: a player in turn order, -1: chance), as arrays in
    breadth-first order. Its shape follows from the two numbers alone."""
    rng = np.random.default_rng([depth, size])
    parent, act, kids, lev = [-1], [-1], [], [0]
    v = 0
    while v < len(parent):
        k = 0
        if lev[v] < depth:
            room = size - len(parent)
            k = int(rng.integers(1, 4)) if lev[v] > 1 else 3
            if lev[v] > 1 and rng.random() < 0.15:
                k = 0
            if k > room:
                k = 0
        kids.append(k)
        for a in range(k):
            parent.append(v)
            act.append(a)
            lev.append(lev[v] + 1)
        v += 1
    kind = rng.integers(0, 10 ** 6, size=len(parent))
    chance = (rng.random(len(parent)) < 0.15) & (np.asarray(kids) > 1)
    return (np.asarray(parent), np.asarray(act), np.asarray(kids), kind, chance)


def _grid(rng, k):
    p = rng.dirichlet(np.ones(k))
    return p / p.sum()


@functools.lru_cache(maxsize=None)
def _public_n(players: int, types: int, depth: int, tree: int) -> Game:
    """A general-sum game: the root deals every player one of ``types`` private types (one chance
    node over all combinations), then the public tree is played; an infoset is (player, own
    type, public node)."""
    tp, ta, kids, kind, chance = _public_tree(depth, tree)
    tn, nd = len(tp), types ** players
    who = np.where(kids == 0, -1, np.where(chance, 0, 1 + kind % players))
    n = 1 + nd * tn
    d = np.repeat(np.arange(nd), tn)
    t = np.tile(np.arange(tn), nd)
    parent = np.concatenate([[-1], np.where(tp[t] < 0, 0, 1 + d * tn + tp[t])])
    action = np.concatenate([[-1], np.where(tp[t] < 0, d, ta[t])])
    # infosets: the deal, then per public node its chance infoset or one per type of its player
    first = np.zeros(tn, dtype=np.int64)
    count = np.where(who < 0, 0, np.where(who == 0, 1, types))
    first[:] = 1 + np.concatenate([[0], np.cumsum(count)[:-1]])
    own = (d // types ** np.maximum(who[t] - 1, 0)) % types
    inf = np.where(who[t] < 0, -1, first[t] + np.where(who[t] == 0, 0, own))
    iplayer = np.concatenate([[0], np.repeat(np.maximum(who, 0), count)])
    inact = np.concatenate([[nd], np.repeat(kids, count)])
    rng = np.random.default_rng(tree)
    cp = [np.full(nd, 1.0 / nd)] + [_grid(rng, int(k)) for k in inact[1:][iplayer[1:] == 0]]
    pay = np.zeros((n, players))
    return Game(name=f"public{players}x{types}x{tn}", parent=parent.astype(np.int32),
                node_infoset=np.concatenate([[0], inf]).astype(np.int32),
                node_action=action.astype(np.int32), infoset_player=iplayer.astype(np.int8),
                infoset_num_actions=inact.astype(np.int32), chance_prob=np.concatenate(cp),
                payoff_u1=pay[:, 0].copy(), payoff_u2=None, payoff=pay)


@functools.lru_cache(maxsize=None)
def _shape(kind: str, *a):
    if kind == "kuhn":
        return games.kuhn_like(*a)
    if kind == "leduc":
        return games.leduc_like(*a)
    if kind == "kuhn3":
        return games.kuhn3(*a, deal="joint")
    if kind == "poker":
        ranks, rounds, cap, stack, deals = a
        return games.poker_game(ranks, rounds, cap, stack, max_deals=deals, scale=True)
    return games.subgame(*a)


def _beliefs(g: Game, rng) -> Game:
    """The game with another distribution at the root's deal (its infoset is the first of the
    chance infosets in every game used here)."""
    h = int(g.node_infoset[0])
    nd = int(g.infoset_num_actions[h])
    p = np.array(g.chance_prob)
    w = 0.05 + rng.random(nd)
    p[:nd] = w / w.sum()
    return dataclasses.replace(g, chance_prob=p)


def _game(case, seed):
    """The case's game, or its list of games, for one seed."""
    rng = np.random.default_rng([seed & 0x7FFFFFFF, 11])
    kind = case["game"]
    if kind == "kuhn":
        return _beliefs(_shape("kuhn", case["ranks"]), rng)
    if kind == "leduc":
        return _beliefs(_shape("leduc", case["ranks"], case["suits"]), rng)
    if kind == "poker":
        return _beliefs(_shape("poker", case["ranks"], case["rounds"], case["cap"], case["stack"],
                               case["deals"]), rng)
    if kind == "batch":
        return [_beliefs(_shape("subgame", s), rng)
                for s in range(case["first"], case["first"] + case["count"])]
    if kind == "kuhn3":
        return _beliefs(_shape("kuhn3", case["ranks"]), rng)
    g = _beliefs(_public_n(case["players"], case["types"], case["depth"], case["tree"]), rng)
    pay = rng.random(g.payoff.shape) * 2.0 - 1.0
    pay[g.node_infoset >= 0] = 0.0
    return dataclasses.replace(g, payoff=pay, payoff_u1=pay[:, 0].copy())


def _start(g, seed):
    """Warm-start regrets, one per infoset-action pair of the game (of each game in turn): of
    the size of an iteration's regrets, all positive."""
    rng = np.random.default_rng([seed & 0x7FFFFFFF, 17])
    got = []
    for x in g if isinstance(g, list) else [g]:
        got.append(1e-3 * (0.1 + np.abs(rng.standard_normal(games.n_player_q(x)))))
    return [r.astype(np.float32).astype(np.float64) for r in got]


# ---------------------------------------------------------------------------- prepare, run


def _desc(rows, rng):
    """Descriptors of ``rows`` poker infosets and the beliefs of 64 games: every field over
    the range that the subgame family gives it."""
    n_games = 64
    d = np.zeros((rows, 16), dtype=np.int16)
    ranks = rng.integers(4, 14, size=rows)
    d[:, 0] = rng.integers(1, 3, size=rows)
    d[:, 1] = rng.integers(0, 13, size=rows) % ranks
    d[:, 2] = rng.integers(0, 3, size=rows)
    for j in range(3):
        d[:, 3 + j] = np.where(d[:, 2] > j, rng.integers(0, 13, size=rows) % ranks, -1)
    d[:, 6] = rng.integers(0, 4, size=rows)
    d[:, 7] = rng.integers(0, 4, size=rows)
    d[:, 10] = rng.choice([20, 60, 150, 400], size=rows)
    d[:, 8] = rng.integers(1, 20, size=rows)
    d[:, 9] = rng.integers(1, 20, size=rows)
    # legal slots: the same masks in another order for another seed (as many pairs in all)
    masks = np.asarray([2 + 4 + 8, 1 + 2 + 4 + 8, 1 + 2, 2 + 8, 1 + 2 + 8])
    d[:, 11] = rng.permutation(np.resize(masks, rows))
    d[:, 12] = rng.integers(0, 16, size=rows)
    d[:, 13] = rng.integers(1, 4, size=rows)
    d[:, 14] = ranks
    d[:, 15] = rng.integers(0, n_games, size=rows)
    bel = rng.dirichlet(np.ones(13), size=(n_games, 2)).astype(np.float32)
    k = sum((d[:, 11].astype(np.int64) >> s) & 1 for s in range(4))
    qoff = np.concatenate([[0], np.cumsum(k)[:-1]]).astype(np.int64)
    return d, bel, qoff, int(k.sum())


def _net_data(case, seed):
    """What the network's calls take, on the host: the same arrays for run and exact."""
    rng = np.random.default_rng([seed & 0x7FFFFFFF, 23])
    rows = case["rows"] * (case["steps"] if case["what"] == "train" else 1)
    desc, bel, qoff, n_q = _desc(rows, rng)
    params = warmstart.he_uniform_params(96, case["hidden"], 4, seed & 0xFFFF)
    return {"desc": desc, "bel": bel, "qoff": qoff, "n_q": n_q, "params": params}


def _features64(desc, bel):
    """The network's inputs in 64 bits (the layout that include/cfr_warmstart.h describes):
    [rows, 96], before they are rounded to bf16."""
    n = len(desc)
    d = desc.astype(np.int64)
    f = np.zeros((n, 96))
    rows = np.arange(n)

    def hot(base, width, col):
        ok = (col >= 0) & (col < width)
        f[rows[ok], base + col[ok]] = 1.0

    hot(0, 13, d[:, 1])
    hot(13, 2, d[:, 0] - 1)
    hot(15, 3, d[:, 2])
    for j in range(3):
        hot(18, 13, d[:, 3 + j])
    hot(31, 4, d[:, 6])
    hot(35, 5, d[:, 7])
    stack, me, op = (d[:, j].astype(np.float64) for j in (10, 8, 9))
    f[:, 40], f[:, 41], f[:, 42] = me / stack, op / stack, (me + op) / stack
    f[:, 43] = (op - me) / np.maximum(me + op, 1.0)
    for s in range(4):
        f[:, 44 + s] = (d[:, 11] >> s) & 1
    f[:, 48], f[:, 49] = d[:, 12] / 16.0, d[:, 13] / 3.0
    f[:, 50], f[:, 51] = np.log(stack) / math.log(1000.0), d[:, 14] / 13.0
    bm = bel[d[:, 15], d[:, 0] - 1].astype(np.float64)
    bo = bel[d[:, 15], 2 - d[:, 0]].astype(np.float64)
    f[:, 52:65], f[:, 65:78] = bo, bm
    r = np.arange(13)[None, :]
    f[:, 78] = (bo * (r < d[:, 1:2])).sum(1)
    f[:, 79] = (bo * (r > d[:, 1:2])).sum(1)
    f[:, 80] = 1.0
    return f


def _targets(case, seed):
    """Training targets: a distribution over each infoset's legal slots, and the legal mask."""
    data = _net_data(case, seed)
    rng = np.random.default_rng([seed & 0x7FFFFFFF, 29])
    legal = ((data["desc"][:, 11:12].astype(np.int64) >> np.arange(4)) & 1).astype(np.float32)
    t = rng.random(legal.shape).astype(np.float32) * legal
    return data, t / t.sum(1, keepdims=True), legal


def prepare(case, seed):
    if case["do"] == "net":
        net = warmstart.WarmStartNet(hidden=case["hidden"], device=DEVICE,
                                     max_batch=8192 if case["what"] == "train" else 65536)
        if case["what"] == "train":
            data, target, legal = _targets(case, seed)
        else:
            data = _net_data(case, seed)
        net.set_params(data["params"])
        dev = {k: torch.from_numpy(data[k]).to(DEVICE) for k in ("desc", "bel", "qoff")}
        state = {"case": case, "net": net, "n_q": data["n_q"], **dev}
        if case["what"] != "predict":
            # the features as the library itself makes them
            state["x"] = warmstart.features(dev["desc"], dev["bel"])
        if case["what"] == "train":
            n = case["rows"]
            cut = [slice(i * n, (i + 1) * n) for i in range(case["steps"])]
            state["batches"] = [(state["x"][c].contiguous(),
                                 torch.from_numpy(target[c]).to(DEVICE),
                                 torch.from_numpy(legal[c]).to(DEVICE)) for c in cut]
        return state
    g = _game(case, seed)
    kw = {"device": DEVICE, "schedule": case["schedule"]}
    if case["game"] == "batch":
        s = BatchSolver(g, case["variant"], **kw)
    elif case["game"] in ("public_n", "kuhn3"):
        s = NPlayerSolver(g, case["variant"], precision=case["precision"], **kw)
    elif case.get("window"):
        s = PartitionedSolver(g, case["variant"], cut_level=case["cut"],
                              max_window_nodes=case["window"], precision=case["precision"], **kw)
    else:
        s = Solver(g, case["variant"], precision=case["precision"], **kw)
    r0 = np.concatenate(_start(g, seed))
    s.set_state(0, r0, np.zeros_like(r0))
    dtype = torch.float64 if case["precision"] == "f64" else torch.float32
    return {"case": case, "solver": s,
            "average": torch.empty(s.n_q, dtype=dtype, device=DEVICE)}


def run(state):
    case = state["case"]
    if case["do"] == "net":
        net = state["net"]
        if case["what"] == "forward":
            return net.forward(state["x"])
        if case["what"] == "predict":
            x = warmstart.features(state["desc"], state["bel"])
            logits = net.forward(x)
            probs = warmstart.probs_to_pairs(logits, state["desc"], state["qoff"], state["n_q"])
            return {"logits": logits, "probs": probs}
        losses = [net.train_step(x, t, m, 1e-3) for x, t, m in state["batches"]]
        return {"losses": np.asarray(losses), "grads": net.grads(), "params": net.params()}
    s = state["solver"]
    s.iterate(case["iters"])
    out = {}
    if case["check"]:
        e = s.exploitability()
        out = {"br1": np.asarray(e["br1"]), "br2": np.asarray(e["br2"])}
    s.average_strategy_device(state["average"])
    out["average"] = state["average"]
    return out


# ------------------------------------------------------------------------------- work


def work(case):
    """Solve: per iteration, each node's structure read once (a 4-byte label per edge), each
    terminal's payoff per player once, and per infoset-action pair the strategy, the regret and
    the strategy sum read and written once; per node a multiply-add each for its value and its
    reach, per pair the update. The average (and the best response, which reads structure, payoffs
    and the average once more) once per pass. Net: each operand read once, each result
    written once, the products of the three layers (three times that for a training step)."""
    if case["do"] == "net":
        rows, h = case["rows"], case["hidden"]
        mac = 96 * h + h * h + h * 4
        if case["what"] == "forward":
            return {"bytes": rows * (2 * 96 + 16) + 2 * mac, "flops": 2 * rows * mac}
        if case["what"] == "predict":
            # descriptors in; logits and about three probabilities out
            return {"bytes": rows * (32 + 8 + 16 + 12) + 2 * mac, "flops": 2 * rows * mac}
        # training: input, target and mask per row; weights, moments and gradient per step
        return {"bytes": case["steps"] * (rows * (2 * 96 + 32) + 4 * 8 * mac),
                "flops": case["steps"] * 6 * rows * mac}
    z = _sizes(case)
    real = 8 if case["precision"] == "f64" else 4
    cols = case.get("players", 3) if case["game"] in ("public_n", "kuhn3") else 1
    tree = 4 * z["nodes"] + real * cols * z["terminals"]
    passes = case["iters"] + (1 if case["check"] else 0)
    return {"bytes": passes * tree + case["iters"] * 6 * real * z["pairs"] + 2 * real * z["pairs"],
            "flops": passes * 4 * cols * z["nodes"] + case["iters"] * 8 * z["pairs"]}


@functools.lru_cache(maxsize=None)
def _sizes_of(*key):
    got = {"nodes": 0, "terminals": 0, "pairs": 0}
    g = _game(dict(key), 1)
    for x in g if isinstance(g, list) else [g]:
        c = x.counts()
        got["nodes"] += c["nodes"]
        got["terminals"] += c["terminals"]
        got["pairs"] += c["infoset_actions"]
    return got


def _sizes(case):
    return _sizes_of(*sorted((k, v) for k, v in case.items() if k not in ("name", "variant")))


# ------------------------------------------------------------------------------- exact


class _Exact:
    """CFR in 64 bits over one game, level by level in plain torch."""

    def __init__(self, g: Game, variant: str, schedule: str, dev):
        T = functools.partial(torch.as_tensor, device=dev)
        par = T(g.parent.astype(np.int64))
        n = par.numel()
        level = torch.zeros(n, dtype=torch.int64, device=dev)
        up = par.clone()
        while True:
            live = up >= 0
            if not bool(live.any()):
                break
            level += live
            up = torch.where(live, par[up.clamp(min=0)], up)
        depth = int(level.max())
        self.levels = [torch.nonzero(level == d).reshape(-1) for d in range(depth + 1)]
        self.par, self.inf, act = par, T(g.node_infoset.astype(np.int64)), T(g.node_action.astype(np.int64))
        ip, nact = T(g.infoset_player.astype(np.int64)), T(g.infoset_num_actions.astype(np.int64))
        rational = ip > 0
        k = torch.where(rational, nact, torch.zeros_like(nact))
        qoff = torch.cumsum(k, 0) - k
        kc = torch.where(rational, torch.zeros_like(nact), nact)
        self.Q = int(k.sum())
        off = torch.where(rational, qoff, self.Q + torch.cumsum(kc, 0) - kc)
        self.P = 2 if g.payoff is None else g.payoff.shape[1]
        ph = self.inf[par.clamp(min=0)]
        # the edge into each node: its index into [sigma | sigma_0], and who acted (0 chance)
        self.edge = torch.where(par >= 0, off[ph] + act, torch.zeros_like(act))
        self.actor = torch.where(par >= 0, ip[ph], torch.zeros_like(act))
        self.sigma0 = T(np.asarray(g.chance_prob, dtype=np.float64))
        term = (self.inf < 0).double()
        pay = (np.stack([g.payoff_u1, -g.payoff_u1], 1) if g.payoff is None else g.payoff)
        self.pay = T(np.asarray(pay, dtype=np.float64)) * term[:, None]
        self.set_of = torch.repeat_interleave(torch.arange(len(ip), device=dev), k)  # pair -> infoset
        self.kq = nact[self.set_of].double()
        self.nh, self.ip = len(ip), ip
        self.R = torch.zeros(self.Q, dtype=torch.float64, device=dev)
        self.S = torch.zeros_like(self.R)
        self.t, self.variant = 0, variant
        everyone = list(range(1, self.P + 1))
        self.passes = [everyone] if schedule == "simultaneous" else [[i] for i in everyone]

    def _share(self, x):
        tot = torch.zeros(self.nh, dtype=torch.float64, device=x.device).index_add_(0, self.set_of, x)[self.set_of]
        return torch.where(tot > 0, x / tot.clamp(min=1e-300), 1.0 / self.kq)

    def iterate(self):
        t = self.t + 1
        for who in self.passes:
            sig = self._share(self.R.clamp(min=0))
            s = torch.cat([sig, self.sigma0])[self.edge]
            n = s.numel()
            reach = torch.ones(n, self.P + 1, dtype=torch.float64, device=s.device)  # chance, players
            for lv in self.levels[1:]:
                r = reach[self.par[lv]]
                r[torch.arange(len(lv), device=s.device), self.actor[lv]] *= s[lv]
                reach[lv] = r
            val = self.pay.clone()
            for lv in reversed(self.levels[1:]):
                val.index_add_(0, self.par[lv], s[lv][:, None] * val[lv])
            R, S = self.R, self.S
            for i in who:
                c = torch.nonzero((self.actor == i) & (self.par >= 0)).reshape(-1)
                p = self.par[c]
                minus = torch.ones(len(c), dtype=torch.float64, device=s.device)
                for j in range(self.P + 1):
                    if j != i:
                        minus = minus * reach[p, j]
                reg = torch.zeros_like(R).index_add_(0, self.edge[c], minus * (val[c, i - 1] - val[p, i - 1]))
                own = torch.zeros_like(R).index_add_(0, self.edge[c], reach[p, i])
                mine = self.ip[self.set_of] == i
                new, add = R + reg, own * sig
                if self.variant == "cfr+":
                    new, avg = new.clamp(min=0), S + t * add
                elif self.variant == "dcfr":
                    f = t ** 1.5 / (t ** 1.5 + 1.0)
                    new = torch.where(new > 0, new * f, new * 0.5)
                    avg = (S + add) * (t / (t + 1.0)) ** 2
                else:
                    avg = S + add
                R, S = torch.where(mine, new, R), torch.where(mine, avg, S)
            self.R, self.S = R, S
        self.t = t

    def average(self):
        return self._share(self.S)

    def best_response(self):
        sig = torch.cat([self.average(), self.sigma0])[self.edge]
        out = []
        for i in (1, 2):
            f = torch.where(self.actor == i, torch.ones_like(sig), sig)
            reach = torch.ones_like(sig)
            for lv in self.levels[1:]:
                reach[lv] = reach[self.par[lv]] * f[lv]
            val = self.pay[:, i - 1].clone()
            for lv in reversed(self.levels[1:]):
                mine = self.actor[lv] == i
                o, c = lv[~mine], lv[mine]
                val.index_add_(0, self.par[o], sig[o] * val[o])
                q = torch.zeros(self.Q, dtype=torch.float64, device=sig.device)
                q.index_add_(0, self.edge[c], reach[self.par[c]] * val[c])
                best = torch.full((self.nh,), -math.inf, dtype=torch.float64, device=sig.device)
                best.scatter_reduce_(0, self.set_of, q, "amax")
                # the first of an infoset's best actions
                idx = torch.arange(self.Q, device=sig.device)
                idx = torch.where(q == best[self.set_of], idx, torch.full_like(idx, self.Q))
                one = torch.full((self.nh,), self.Q, dtype=torch.int64, device=sig.device)
                one.scatter_reduce_(0, self.set_of, idx, "amin")
                take = c[self.edge[c] == one[self.inf[self.par[c]]]]
                val[self.par[take]] = val[take]
            out.append(float(val[self.levels[0][0]]))
        return out


def exact(case, seed):
    dev = DEVICE if torch.cuda.is_available() else "cpu"
    if case["do"] == "net":
        return _exact_net(case, seed, dev)
    g = _game(case, seed)
    many = isinstance(g, list)
    avg, br = [], []
    for x, r0 in zip(g if many else [g], _start(g, seed)):
        e = _Exact(x, case["variant"], case["schedule"], dev)
        e.R = torch.from_numpy(r0).to(dev)
        for _ in range(case["iters"]):
            e.iterate()
        avg.append(e.average().cpu())
        if case["check"]:
            br.append(e.best_response())
    out = {"average": torch.cat(avg)}
    if case["check"]:
        b = np.asarray(br)
        out["br1"], out["br2"] = (b[:, 0], b[:, 1]) if many else (b[0, 0], b[0, 1])
    return out


def _exact_net(case, seed, dev):
    if case["what"] == "train":
        # Adam's steps follow the signs of gradients that rounding decides: no 64-bit value
        return None
    data = _net_data(case, seed)
    h = case["hidden"]
    x = torch.from_numpy(_features64(data["desc"], data["bel"])).to(dev)
    w = torch.from_numpy(data["params"]).to(dev).double()
    at = np.cumsum([0, 96 * h, h, h * h, h, h * 4, 4])
    w1, b1, w2, b2, w3, b3 = (w[a:b] for a, b in zip(at[:-1], at[1:]))
    z = torch.relu(x @ w1.reshape(96, h) + b1)
    z = torch.relu(z @ w2.reshape(h, h) + b2) @ w3.reshape(h, 4) + b3
    if case["what"] == "forward":
        return z
    legal = ((torch.from_numpy(data["desc"][:, 11].astype(np.int64)).to(dev)[:, None]
              >> torch.arange(4, device=dev)) & 1).bool()
    p = torch.softmax(z.masked_fill(~legal, -math.inf), 1)
    return {"logits": z, "probs": p[legal]}
