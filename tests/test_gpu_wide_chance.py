"""Chance nodes of more children than a wavefront has lanes: an iteration's one launch sums them in the
order of the public-block engine's launches (graph=False), so that they agree bit for bit, their own
values and whatever those feed."""
import numpy as np
import pytest

import games
from games.tuple import GameBuilder

pytestmark = pytest.mark.gpu


def _below_player(fan, types, seed=11):
    """Player 1 picks one of three chance nodes of `fan` outcomes each, of which player 2 sees a type;
    both act once more, so that the chance values enter player 1's regrets at the root (no infoset
    is larger than a chunk of the level launches, whose order is their shape's)."""
    rng = np.random.default_rng(seed)
    b = GameBuilder(f"below{fan}")
    root = b.node(-1, -1)
    b.decide(root, b.infoset_id("root", 1, 3))
    for i in range(3):
        c = b.node(root, i)
        w = rng.integers(1, 8, size=fan)
        b.decide(c, b.infoset_id(("c", i), 0, fan, list(w / w.sum())))
        for o in range(fan):
            x = b.node(c, o)
            b.decide(x, b.infoset_id(("p2", i, o % types), 2, 2))
            for a in range(2):
                y = b.node(x, a)
                b.decide(y, b.infoset_id(("p1", i, a, o % (types + 3)), 1, 2))
                for d in range(2):
                    b.terminal(b.node(y, d), float(rng.integers(-64, 65)) / 64)
    return b.build()


# one workgroup; teams of them
GAMES = {
    "65": lambda: _below_player(65, 5),
    "257": lambda: _below_player(257, 7),
    "300": lambda: _below_player(300, 12),
    "4095": lambda: _below_player(4095, 50),
    "root_1190": lambda: games.kuhn_like(35, "joint"),
}


@pytest.mark.parametrize("variant,schedule", [("cfr+", "simultaneous"), ("dcfr", "alternating")])
@pytest.mark.parametrize("name", sorted(GAMES))
def test_bit_for_bit(name, variant, schedule):
    from paper_2408_14778_amd import BatchSolver, Solver
    g = GAMES[name]()
    T, R, S = games.random_state(g, seed=3, nonnegative=variant == "cfr+")
    R, S = R.astype(np.float32), S.astype(np.float32)
    a = Solver(g, variant, schedule=schedule)
    b = Solver(g, variant, schedule=schedule, graph=False)
    assert a.info["engine"] == 1
    dec = a.layout("node_player") >= 0
    for s in (a, b):
        s.set_state(T, R, S)
    for n in (1, 3):
        for s in (a, b):
            s.iterate(n)
        for x, y in zip(a.get_state(), b.get_state()):
            assert np.array_equal(x, y)
        (ua, ra), (ub, rb) = a.node_values(), b.node_values()
        assert np.array_equal(ua, ub) and np.array_equal(ra[dec], rb[dec])
    many = [BatchSolver([g, games.kuhn_like(3, "joint")], variant, schedule=schedule, graph=graph)
            for graph in (True, False)]
    for m in many:
        m.iterate(4)
    for x, y in zip(many[0].get_state(), many[1].get_state()):
        assert np.array_equal(x, y)
