"""Destroying a solver, a batch or a network waits for its own stream alone, not for what other streams
run; the pinned words that they held are used again."""
import pytest

import games

pytestmark = pytest.mark.gpu


def _solver():
    from paper_2408_14778_amd import Solver
    s = Solver(games.leduc_like(3, 2, deal="joint"), "cfr+")
    s.iterate(3)
    s.exploitability()
    return s


def _batch():
    from paper_2408_14778_amd import BatchSolver
    s = BatchSolver([games.kuhn_like(3, "joint"), games.rock_paper_scissors()], "cfr+")
    s.iterate(3)
    s.exploitability()
    return s


def _net():
    from paper_2408_14778_amd.warmstart import WarmStartNet
    return WarmStartNet(96, 64, 4, max_batch=32)


@pytest.mark.parametrize("make", [_solver, _batch, _net])
def test_other_streams_go_on(make):
    import torch
    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    (a @ a)
    other = torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(2):
        s = make()
        torch.cuda.synchronize()
        with torch.cuda.stream(other):
            for _ in range(200):  # about 150 ms
                a @ a
            done = torch.cuda.Event()
            done.record(other)
        s.close()
        assert not done.query()
        torch.cuda.synchronize()


def test_many_solvers_have_words_of_their_own():
    """More than the words of one line, given back and taken again in another order."""
    from paper_2408_14778_amd import BatchSolver, Solver
    small = [games.kuhn_like(r, "joint") for r in (3, 4, 5)]
    want = []
    for g in small:
        s = Solver(g, "cfr+")
        s.iterate(11)
        want.append(s.exploitability()["expl"])
        s.close()
    batch = BatchSolver([small[i % 3] for i in range(40)], "cfr+")
    solvers = [Solver(small[i % 3], "cfr+") for i in range(40)]
    for s in solvers[::2]:
        s.close()
    again = [Solver(g, "cfr+") for g in small]
    batch.iterate(11)
    for i, s in [(i, s) for i, s in enumerate(solvers) if i % 2] + list(enumerate(again)):
        s.iterate(11)
        assert s.exploitability()["expl"] == want[i % 3]
    assert [float(x) for x in batch.exploitability()["expl"]] == [want[i % 3] for i in range(40)]
