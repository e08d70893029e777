"""A call of many iterations is several launches of bounded length (each forms its team anew), with the
results of the same iterations call by call."""
import numpy as np
import pytest

import games

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("schedule", ["simultaneous", "alternating"])
@pytest.mark.parametrize("make", [lambda: games.kuhn_like(3, "joint"),
                                  lambda: games.poker_game(10, 3, 1, 60, max_deals=31)],
                         ids=["one_workgroup", "team"])
def test_launches_of_a_call(make, schedule):
    from paper_2408_14778_amd import Solver
    g = make()
    a, b = (Solver(g, "cfr+", schedule=schedule) for _ in range(2))
    most = int(a.layout("one_launch")[3])
    passes = 2 if schedule == "alternating" else 1
    # about 5 ms at 4 us an iteration and 22 ps a node and pass
    assert 16 <= most and most * (4 + 22e-6 * g.n_nodes * passes) <= 5000
    a.iterate(2 * most + 3)
    for n in (1, most, most - 1, 3):
        b.iterate(n)
    for x, y in zip(a.get_state(), b.get_state()):
        assert np.array_equal(x, y)
    for x, y in zip(a.node_values(), b.node_values()):
        assert np.array_equal(x, y)
