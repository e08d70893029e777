"""Batches whose iterations run in one launch against the level-by-level launches of the same batch
(graph=False), bit for bit: a forest in one workgroup, in a team of them, a batch of one game, and
games of different depths."""
import numpy as np
import pytest

import games

pytestmark = pytest.mark.gpu

BATCHES = {
    "one_workgroup": lambda: [games.kuhn_like(3, "joint"), games.rock_paper_scissors()],
    "one_game": lambda: [games.leduc_like(3, 2, deal="sequential")],
    "depths": lambda: [games.random_game(66, deal="sequential", depth=30, max_actions=2, p_terminal=0.3),
                       games.kuhn_like(20, "joint"), games.random_game(5, deal="none", depth=7)],
    "sixteen_actions": lambda: [games.random_game(72, deal="joint", depth=3, max_actions=16),
                                games.leduc_like(4, 2, deal="joint")],
    "subgames": lambda: [games.subgame(s) for s in (102, 103, 104, 109, 111)],
}


@pytest.mark.parametrize("schedule", ["simultaneous", "alternating"])
@pytest.mark.parametrize("variant", ["vanilla", "cfr+", "dcfr"])
@pytest.mark.parametrize("name", sorted(BATCHES))
def test_forest_bit_for_bit(name, variant, schedule):
    from paper_2408_14778_amd import BatchSolver
    batch = BATCHES[name]()
    a = BatchSolver(batch, variant, schedule=schedule)
    b = BatchSolver(batch, variant, schedule=schedule, graph=False)
    states = [games.random_state(g, seed=5 + i, nonnegative=variant == "cfr+")
              for i, g in enumerate(batch)]
    R = np.concatenate([x[1] for x in states]).astype(np.float32)
    S = np.concatenate([x[2] for x in states]).astype(np.float32)
    for s in (a, b):
        s.set_state(37, R, S)
    for n in (1, 3):
        a.iterate(n)
        for _ in range(n):
            b.iterate(1)
        for x, y in zip(a.get_state(), b.get_state()):
            assert np.array_equal(x, y), (name, n)
        ea, eb = a.exploitability(), b.exploitability()
        assert np.array_equal(np.asarray(ea["expl"]), np.asarray(eb["expl"]))
    a.close()
    b.close()
