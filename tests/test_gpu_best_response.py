"""Best responses of the node engine and the public-block engine at their branches: reach by walks to
the root or level by level (more than 24 levels), more actions than a walk over the members takes,
member counts off the walks' width, a root wider than a wavefront, a single node.

The tolerance: a value is a convex combination over at most D levels of at most K children, each
level rounding by at most (K + 4) units of the largest payoff, and the choice at an infoset compares
sums over at most m members; an action chosen wrongly within that rounding loses no more than it."""
import numpy as np
import pytest

import games
from oracle import br, cfr
from oracle.tree import Tree

pytestmark = pytest.mark.gpu

GAMES = {
    "deep": lambda: games.random_game(66, deal="sequential", depth=30, max_actions=2, p_terminal=0.3),
    "sixteen_actions": lambda: games.random_game(72, deal="joint", depth=3, max_actions=16),
    "no_chance": lambda: games.random_game(5, deal="none", depth=7),
    "wide_root": lambda: games.kuhn_like(35, "joint"),
    "poker": lambda: games.poker_game(7, 2, 2, 60, max_deals=41),
}


@pytest.mark.parametrize("engine", ["auto", "node", "f64"])
@pytest.mark.parametrize("name", sorted(GAMES))
def test_best_response_values(name, engine):
    from paper_2408_14778_amd import Solver
    g = GAMES[name]()
    f64 = engine == "f64"
    t = Tree(g)
    s = Solver(g, "cfr+", precision="f64") if f64 else Solver(g, "cfr+", engine=engine)
    K = max(len(c) for c in t.children)
    members = max(len(m) for m in t.members.values())
    depth = s.info["depth"]
    for seed in (3, 4):  # (the second on the arrays that the first left behind)
        T, R, S = games.random_state(g, seed=seed, nonnegative=True)
        s.set_state(T, R.astype(np.float64 if f64 else np.float32),
                    S.astype(np.float64 if f64 else np.float32))
        got = s.exploitability()
        ref = br.exploitability(t, cfr.average_strategy(t, [float(x) for x in S]))
        tol = (depth * (K + 4) + members) * 2.0 ** (-53 if f64 else -24) * max(map(abs, t.u1))
        assert abs(got["expl"] - ref["expl"]) <= tol, (got, ref, tol)
    s.close()
