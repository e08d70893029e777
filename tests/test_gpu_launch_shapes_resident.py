"""Launch shapes on solvers whose iterations are one launch: asking for shapes makes them launches of
those shapes (a captured graph of them), the defaults return the one launch, and nothing else
changes."""
import numpy as np
import pytest

import games

pytestmark = pytest.mark.gpu


def _single(**kw):
    from paper_2408_14778_amd import Solver
    return Solver(games.leduc_like(4, 2, deal="sequential"), "cfr+", **kw)


def _batch(**kw):
    from paper_2408_14778_amd import BatchSolver
    return BatchSolver([games.leduc_like(3, 2, deal="joint"), games.kuhn_like(3, "joint")], "cfr+", **kw)


@pytest.mark.parametrize("make", [_single, _batch], ids=["game", "batch"])
@pytest.mark.parametrize("graph", [True, False])
def test_shapes_take_effect(make, graph):
    ref = make()
    assert ref.one_launch  # the tuned shapes, which constructors apply, leave it so
    s = make(graph=graph)
    assert s.one_launch == graph
    ref.iterate(9)
    s.iterate(2)
    s.set_launch_shape(up_threads=64, up_members=1, reach_threads=64, reach_nodes=1)
    assert not s.one_launch and not s.layout("one_launch").any()
    s.iterate(3)
    if make is _single:  # the values are the last iteration's, whichever launches ran it
        five = make()
        five.iterate(5)
        dec = s.layout("node_player") >= 0
        (ua, ra), (ub, rb) = s.node_values(), five.node_values()
        assert np.array_equal(ua, ub) and np.array_equal(ra[dec], rb[dec])
    s.set_launch_shape(up_threads=512, up_members=2, reach_threads=1024, reach_nodes=2)
    s.iterate(1)
    s.set_launch_shape()
    assert s.one_launch == graph
    s.iterate(3)
    for x, y in zip(s.get_state(), ref.get_state()):
        assert np.array_equal(x, y)
