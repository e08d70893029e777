"""The out-of-core iteration where its second cut matters: subtrees larger than a workgroup takes (so
that levels lie between the two cuts), several groups of partitions, runs of one and of many
subtrees, against the in-core node engine from the same seeded state.

Tolerances are those of the partitioned iteration's other tests: both sides sum the same terms in
another order, 1e-6 (double precision 1e-12) norm-wise."""
import numpy as np
import pytest

import games

pytestmark = pytest.mark.gpu


def _uneven():
    """A root dealing 100 ways to nodes of 60 actions; under the first of them every action leads to
    a node of 40 more. The first subtree is larger than a run, and the nodes between the cuts are
    more than its partition's: three groups."""
    deals, wide, deep = 100, 60, 40
    parent, infoset, action, payoff = [-1], [0], [-1], [0.0]
    players, k = [0], [deals]
    rng = np.random.default_rng(11)

    def add(p, a, h, u=0.0):
        parent.append(p)
        action.append(a)
        infoset.append(h)
        payoff.append(u)
        return len(parent) - 1

    tops = []
    for d in range(deals):
        players.append(1)
        k.append(wide)
        tops.append(add(0, d, len(players) - 1))
    players.append(2)
    k.append(deep)
    below = len(players) - 1
    for d, top in enumerate(tops):
        for a in range(wide):
            if d > 0:
                add(top, a, -1, rng.uniform(-1, 1))
                continue
            v = add(top, a, below)
            for b in range(deep):
                add(v, b, -1, rng.uniform(-1, 1))
    return games.Game("uneven", np.array(parent, np.int32), np.array(infoset, np.int32),
                      np.array(action, np.int32), np.array(players, np.int8), np.array(k, np.int32),
                      np.full(deals, 1.0 / deals), np.array(payoff))


GAMES = {
    "uneven": (_uneven, (1, 2)),
    "leduc6x2": (lambda: games.leduc_like(6, 2, deal="joint"), (1, 3)),
    "poker": (lambda: games.poker_game(7, 2, 2, 60, max_deals=5), (1, 2, 5)),
}


@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("name", sorted(GAMES))
def test_second_cut(name, precision):
    from paper_2408_14778_amd import PartitionedSolver, Solver
    make, cuts = GAMES[name]
    g = make()
    real, tol = (np.float64, 1e-12) if precision == "f64" else (np.float32, 1e-6)
    T, R, S = games.random_state(g, seed=17)
    ref = Solver(g, "dcfr", engine="node", precision=precision, graph=False)
    ref.set_state(T, R.astype(real), S.astype(real))
    ref.iterate(1)
    want = ref.get_state()
    for cut in cuts:
        for window in (1, 700, 1 << 40):
            s = PartitionedSolver(g, "dcfr", cut_level=cut, max_window_nodes=window,
                                  precision=precision)
            s.set_state(T, R.astype(real), S.astype(real))
            s.iterate(1)
            got = s.get_state()
            assert got[0] == want[0]
            for a, b in zip(got[1:], want[1:]):
                assert np.abs(a - b).max() <= tol * np.abs(b).max(), (cut, window)
            s.close()
    ref.close()
