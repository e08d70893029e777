"""Whole iterations in one launch against the level-by-level launches of the same solver
(graph=False): a game in one workgroup, a team of workgroups on one XCD, a team over the chip, and
workgroups that take several bins, in both precisions, for every variant and schedule, and for
general-sum games."""
import dataclasses

import numpy as np
import pytest

import games

pytestmark = pytest.mark.gpu

# two players: one workgroup (also at its largest, and without chance), one XCD (a 1,190-way root,
# wider than the lanes of a wavefront; chance inside the subtrees; deep sequential deals), the chip
TWO = {
    "one_terminal_deep": lambda: games.random_game(66, deal="sequential", depth=30, max_actions=2,
                                                   p_terminal=0.3),
    "solo": lambda: games.kuhn_like(3, "joint"),
    "solo_no_chance": lambda: games.random_game(5, deal="none", depth=7),
    "solo_16_actions": lambda: games.random_game(72, deal="joint", depth=3, max_actions=16),
    "team_wide_root": lambda: games.kuhn_like(35, "joint"),
    "team": lambda: games.leduc_like(4, 2, deal="sequential"),
    "team_odd": lambda: games.poker_game(7, 2, 2, 60, max_deals=41),
    "chip": lambda: games.poker_game(10, 3, 1, 60, max_deals=31),
}
_cache = {}


def _game(name):
    if name not in _cache:
        _cache[name] = TWO[name]()
    return _cache[name]


def _state(g, seed, real, variant):
    T, R, S = games.random_state(g, seed=seed, nonnegative=variant == "cfr+")
    return T, R.astype(real), S.astype(real)


@pytest.mark.parametrize("schedule", ["simultaneous", "alternating"])
@pytest.mark.parametrize("variant", ["vanilla", "cfr+", "dcfr"])
@pytest.mark.parametrize("name", sorted(TWO))
def test_single_precision_bit_for_bit(name, variant, schedule):
    """The public-block engine's launches sum in the same order: state, strategy and node values
    agree bit for bit after one iteration and after more, whatever the calls they come in."""
    from paper_2408_14778_amd import Solver
    g = _game(name)
    a = Solver(g, variant, schedule=schedule)
    b = Solver(g, variant, schedule=schedule, graph=False)
    st = _state(g, 3, np.float32, variant)
    dec = a.layout("node_player") >= 0
    # (the two agree where the engine they are compared with sums without atomics)
    exact = a.info["engine"] == 1
    for s in (a, b):
        s.set_state(*st)
    for n in (1, 3):
        a.iterate(n)
        for _ in range(n):
            b.iterate(1)
        (Ta, Ra, Sa), (Tb, Rb, Sb) = a.get_state(), b.get_state()
        assert Ta == Tb
        (ua, ra), (ub, rb) = a.node_values(), b.node_values()
        pairs = [(Ra, Rb), (Sa, Sb), (a.current_strategy(), b.current_strategy()),
                 (ra[dec], rb[dec]), (ua[1:], ub[1:])]
        for x, y in pairs:
            if exact:
                assert np.array_equal(x, y)
            else:
                np.testing.assert_allclose(x, y, rtol=1e-4, atol=1e-5)
        # the root's value: a 1,190-way sum in another order
        assert abs(ua[0] - ub[0]) <= 2e-6 * max(1.0, np.abs(ub).max())
    assert a.exploitability() == b.exploitability() or not exact


@pytest.mark.parametrize("name", ["solo", "team_wide_root", "team", "chip"])
@pytest.mark.parametrize("variant", ["cfr+", "dcfr"])
def test_double_precision(name, variant):
    """Against the node engine's launches, whose atomics add in any order: a few roundings of 2^-53
    per sum of at most a few hundred terms."""
    from paper_2408_14778_amd import Solver
    g = _game(name)
    a = Solver(g, variant, precision="f64")
    b = Solver(g, variant, precision="f64", graph=False)
    st = _state(g, 4, np.float64, variant)
    for s in (a, b):
        s.set_state(*st)
        s.iterate(2)
    (_, Ra, Sa), (_, Rb, Sb) = a.get_state(), b.get_state()
    for x, y in ((Ra, Rb), (Sa, Sb), *zip(a.node_values(), b.node_values())):
        dec = a.layout("node_player") >= 0
        if x.ndim == 2:
            x, y = x[dec], y[dec]
        assert np.abs(x - y).max() <= 1e-12 * np.abs(y).max()


def _public_n(players, types, depth, seed):
    return games.random_game_n(seed, n_players=players, n_types=types, depth=depth)


# players, types, depth, seed: one workgroup, a team, eight players (as many value columns)
@pytest.mark.parametrize("players,types,depth,seed", [(3, 2, 4, 1), (3, 6, 6, 2), (8, 2, 4, 3)])
@pytest.mark.parametrize("schedule", ["simultaneous", "alternating"])
@pytest.mark.parametrize("precision,tol", [("f32", 2e-5), ("f64", 1e-12)])
def test_general_sum(players, types, depth, seed, schedule, precision, tol):
    """Sums of up to a few hundred members in another order (2^-24 or 2^-53 each), over two
    iterations."""
    from paper_2408_14778_amd import NPlayerSolver
    g = _public_n(players, types, depth, seed)
    real = np.float32 if precision == "f32" else np.float64
    a = NPlayerSolver(g, "cfr+", precision=precision, schedule=schedule)
    b = NPlayerSolver(g, "cfr+", precision=precision, schedule=schedule, graph=False)
    st = _state(g, 6, real, "cfr+")
    for s in (a, b):
        s.set_state(*st)
        s.iterate(2)
    (_, Ra, Sa), (_, Rb, Sb) = a.get_state(), b.get_state()
    dec = a.layout("node_player") >= 0
    (ua, ra), (ub, rb) = a.node_values(), b.node_values()
    for x, y in ((Ra, Rb), (Sa, Sb), (ua, ub), (ra[dec], rb[dec])):
        if x.size:
            assert np.abs(x - y).max() <= tol * max(1e-30, np.abs(y).max())


@pytest.mark.parametrize("deals,precision", [(16, "f64"), (24, "f32")])
def test_several_bins_per_workgroup(deals, precision):
    """Games past one bin per workgroup (2.2 and 3.3 million nodes)."""
    from paper_2408_14778_amd import Solver
    g = games.poker_game(13, 3, 3, 400, max_deals=deals)
    real = np.float32 if precision == "f32" else np.float64
    a = Solver(g, "cfr+", precision=precision)
    b = Solver(g, "cfr+", precision=precision, graph=False)
    st = _state(g, 8, real, "cfr+")
    for s in (a, b):
        s.set_state(*st)
        s.iterate(2)
    (_, Ra, Sa), (_, Rb, Sb) = a.get_state(), b.get_state()
    if precision == "f32":
        assert np.array_equal(Ra, Rb) and np.array_equal(Sa, Sb)
    else:
        for x, y in ((Ra, Rb), (Sa, Sb)):
            assert np.abs(x - y).max() <= 1e-12 * np.abs(y).max()


def test_calls_mix_with_timed_and_restored_iterations():
    """Timed iterations run level by level and share the state; a restored state repeats; solvers
    on several streams do not disturb one another."""
    import torch
    from paper_2408_14778_amd import Solver
    g = _game("team")
    st = _state(g, 9, np.float32, "cfr+")
    ref = Solver(g, "cfr+", graph=False)
    ref.set_state(*st)
    ref.iterate(7)
    want = ref.get_state()
    s = Solver(g, "cfr+")
    for _ in range(2):
        s.set_state(*st)
        s.iterate(3)
        s.iterate_timed(2)
        assert s.node_values()[0].shape == (g.n_nodes,)
        s.iterate(2)
        got = s.get_state()
        assert got[0] == want[0]
        assert np.array_equal(got[1], want[1]) and np.array_equal(got[2], want[2])
    streams = [torch.cuda.Stream() for _ in range(3)]
    many = [Solver(g, "cfr+", stream=st_) for st_ in streams]
    for m in many:
        m.set_state(*st)
    torch.cuda.synchronize()
    for m in many:  # in flight together: the teams form from what is running
        m.iterate(7)
    torch.cuda.synchronize()
    for m in many:
        got = m.get_state()
        assert np.array_equal(got[1], want[1]) and np.array_equal(got[2], want[2])
