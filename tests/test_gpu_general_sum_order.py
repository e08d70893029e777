"""General-sum games give the same bits on every run, whatever launches compute them: whole iterations
in one launch against the level-by-level launches (graph=False, and timed iterations), over every order
of sums that the level and infoset sizes choose."""
import numpy as np
import pytest

import games
from games.tuple import GameBuilder

pytestmark = pytest.mark.gpu


def _uneven(seed=5):
    """Chance nodes of 100, 70 and 2 children on levels of 3 (wavefronts in order), 300 (a butterfly)
    and 21,000 nodes (child order); one player sees only the first deal (14,000 members per
    infoset, among infosets of 1), in a game whose mean infoset is small."""
    rng = np.random.default_rng(seed)
    b = GameBuilder("uneven_n3")

    def deal(v, key, k):
        w = rng.integers(1, 8, size=k)
        b.decide(v, b.infoset_id(("c",) + key, 0, k, list(w / w.sum())))
        return [b.node(v, a) for a in range(k)]

    root = b.node(-1, -1)
    for i, x in enumerate(deal(root, (), 3)):
        for j, y in enumerate(deal(x, (i,), 100)):
            for k, z in enumerate(deal(y, (i, j), 70)):
                for m, d in enumerate(deal(z, (i, j, k), 2)):
                    if (j + k) % 5:
                        b.terminal_vec(d, [float(t) / 64 for t in rng.integers(-64, 65, size=3)])
                        continue
                    who, key = (1, ("a", i)) if m else (2 + k % 2, (i, j, k))
                    b.decide(d, b.infoset_id(key, who, 3))
                    for a in range(3):
                        b.terminal_vec(b.node(d, a),
                                       [float(t) / 64 for t in rng.integers(-64, 65, size=3)])
    return b.build(players=3)


# one workgroup; roots of 8, 64, 343, 729 and 1,728 children, infosets of 4 to 144 members (gathers
# of one, two and four wavefronts); eight players; up to 16 actions, and single ones
GAMES = {
    "kuhn": lambda: games.kuhn3(),
    "types2": lambda: games.random_game_n(1, 3, 2, 4),
    "types4": lambda: games.random_game_n(5, 3, 4, 6),
    "types7": lambda: games.random_game_n(4, 3, 7, 5),
    "types9": lambda: games.random_game_n(3, 3, 9, 5),
    "types12": lambda: games.random_game_n(6, 3, 12, 6, p_terminal=0.15),
    "eight": lambda: games.random_game_n(3, 8, 2, 4),
    "sixteen_actions": lambda: games.random_game_n(8, 2, 5, 3, max_actions=16),
    "one_action": lambda: games.random_game_n(9, 2, 30, 4, max_actions=1, p_chance=0.0),
    "uneven": _uneven,
}
_cache = {}


@pytest.mark.parametrize("schedule", ["simultaneous", "alternating"])
@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("name", sorted(GAMES))
def test_same_bits_on_every_route(name, precision, schedule):
    from paper_2408_14778_amd import NPlayerSolver
    if name not in _cache:
        _cache[name] = GAMES[name]()
    g = _cache[name]
    T, R, S = games.random_state(g, seed=6, nonnegative=True)
    real = np.float32 if precision == "f32" else np.float64
    a = NPlayerSolver(g, "cfr+", precision=precision, schedule=schedule)
    b = NPlayerSolver(g, "cfr+", precision=precision, schedule=schedule, graph=False)
    c = NPlayerSolver(g, "cfr+", precision=precision, schedule=schedule)
    dec = a.layout("node_player") >= 0
    for s in (a, b, c):
        s.set_state(T, R.astype(real), S.astype(real))
    for n in (1, 3):
        a.iterate(n)
        b.iterate(n)
        c.iterate_timed(n)
        (ua, ra), (ub, rb) = a.node_values(), b.node_values()
        assert np.array_equal(ua, ub) and np.array_equal(ra[dec], rb[dec])
        for s in (b, c):
            for x, y in zip(a.get_state(), s.get_state()):
                assert np.array_equal(x, y)
