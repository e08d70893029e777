"""Which way a solver iterates, asserted where it matters: the one launch in each of its shapes (one
workgroup, a team on one XCD, over the chip, several bins per workgroup, a team smaller than
planned), and the level-by-level launches, which small games no longer take by themselves, under
the tests that are about them."""
import numpy as np
import pytest

import games
import test_gpu_branches as branches
import test_gpu_fp64 as fp64
import test_gpu_nplayer as nplayer
import test_gpu_parity as parity
import test_gpu_resident as resident
import test_gpu_warmstart_fused as fused

pytestmark = pytest.mark.gpu

SHAPE = {"one_terminal_deep": "xcd", "solo": "solo", "solo_no_chance": "solo",
         "solo_16_actions": "solo", "team_wide_root": "xcd", "team": "xcd", "team_odd": "xcd", "chip": "chip"}


def _shape(s):
    on, workgroups, bins, _ = (int(x) for x in s.layout("one_launch"))
    assert on == 1
    return "solo" if workgroups == 1 else "xcd" if workgroups <= 32 else "chip", workgroups, bins


def _limit(s, workgroups):
    assert s._lib.cfr_internal_limit_team(s._h, workgroups) == 0
    assert s.layout("one_launch")[1] == min(workgroups, s.layout("one_launch")[2])


@pytest.mark.parametrize("name", sorted(resident.TWO))
@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_shape_of_the_one_launch(name, precision):
    from paper_2408_14778_amd import Solver
    s = Solver(resident._game(name), "cfr+", precision=precision)
    shape, workgroups, bins = _shape(s)
    print(name, precision, shape, workgroups, bins, flush=True)
    assert workgroups == min(bins, 256)
    if precision == "f32":
        assert shape == SHAPE[name]


@pytest.mark.parametrize("workgroups", [1, 2, 3, 9])
@pytest.mark.parametrize("variant,schedule", [("cfr+", "alternating"), ("dcfr", "simultaneous"),
                                              ("vanilla", "alternating")])
@pytest.mark.parametrize("name", ["team_wide_root", "team_odd", "chip"])
def test_smaller_teams_bit_for_bit(name, variant, schedule, workgroups):
    """Bins taken in turn and reloaded, the trunk by a workgroup of its own or by the only one."""
    from paper_2408_14778_amd import Solver
    g = resident._game(name)
    st = resident._state(g, 3, np.float32, variant)
    a = Solver(g, variant, schedule=schedule)
    b = Solver(g, variant, schedule=schedule, graph=False)
    assert b.layout("one_launch")[0] == 0 and a.info["engine"] == 1
    _limit(a, workgroups)
    for s in (a, b):
        s.set_state(*st)
        s.iterate(3)
    for x, y in zip((*a.get_state(), a.node_values()[0]), (*b.get_state(), b.node_values()[0])):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("workgroups", [1, 2, 5, 40])
@pytest.mark.parametrize("schedule", ["simultaneous", "alternating"])
@pytest.mark.parametrize("players", [2, 3])
def test_smaller_teams_in_double_precision_and_general_sums(players, schedule, workgroups):
    """The sums' order does not depend on the team."""
    from paper_2408_14778_amd import NPlayerSolver, Solver
    if players == 2:
        g, kw = resident._game("chip"), dict(precision="f64")
        make = Solver
    else:
        g, kw = games.random_game_n(6, 3, 12, 6, p_terminal=0.15), {}
        make = NPlayerSolver
    a, b = (make(g, "dcfr", schedule=schedule, **kw) for _ in range(2))
    assert _shape(a)[0] == "chip"
    _limit(a, workgroups)
    for s in (a, b):
        s.iterate(4)
    for x, y in zip((*a.get_state(), *a.node_values()), (*b.get_state(), *b.node_values())):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("variant,schedule", [("dcfr", "simultaneous"), ("cfr+", "alternating")])
def test_several_bins_per_workgroup(variant, schedule):
    """As planned (3.3 million nodes), for the variants beside simultaneous CFR+."""
    from paper_2408_14778_amd import Solver
    g = games.poker_game(13, 3, 3, 400, max_deals=24)
    a = Solver(g, variant, schedule=schedule)
    b = Solver(g, variant, schedule=schedule, graph=False)
    shape, workgroups, bins = _shape(a)
    assert shape == "chip" and workgroups == 256 and bins > 256
    st = resident._state(g, 8, np.float32, variant)
    for s in (a, b):
        s.set_state(*st)
        s.iterate(2)
    for x, y in zip(a.get_state(), b.get_state()):
        assert np.array_equal(x, y)


# ---- the level-by-level launches, under the tests that are about them

def _by_level(monkeypatch, module, **more):
    """module._solver makes solvers that run their launches level by level."""
    make = module._solver

    def solver(*args, **kw):
        s = make(*args, **{**kw, **more})
        assert not (s[1] if isinstance(s, tuple) else s).layout("one_launch").any()
        return s
    monkeypatch.setattr(module, "_solver", solver)


@pytest.mark.parametrize("module", [parity, fp64], ids=["f32", "f64"])
def test_graph_replay_matches_direct_launches(monkeypatch, module):
    """keep_node_values asks for level-by-level launches, replayed as a captured graph."""
    _by_level(monkeypatch, module, keep_node_values=True)
    if module is parity:
        parity.test_graph_replay_matches_direct_launches("auto")
    else:
        fp64.test_fp64_graph_replay_matches_direct_launches()


@pytest.mark.parametrize("name", sorted(branches.GAMES))
def test_wide_and_big_infosets(monkeypatch, name):
    _by_level(monkeypatch, branches, keep_node_values=True)
    branches.test_best_response_on_wide_and_big_infosets(name)
    iters = {"matrix7x9": 1000, "rand_wide": 400}.get(name, 200)
    branches.test_exploitability_after_T_on_wide_and_big_infosets(name, "cfr+", iters)


def _by_level_n(g, variant, precision, schedule="simultaneous"):
    from paper_2408_14778_amd import NPlayerSolver
    s = NPlayerSolver(g, variant, precision=precision, schedule=schedule, graph=False)
    assert not s.one_launch
    return s


@pytest.mark.parametrize("precision,tol", [("f32", 1e-6), ("f64", 1e-12)])
@pytest.mark.parametrize("name", sorted(nplayer.GAMES))
def test_general_sum_launches(monkeypatch, name, precision, tol):
    """The general-sum level kernels (gathers of one and two wavefronts) against the oracle."""
    monkeypatch.setattr(nplayer, "_solver", _by_level_n)
    for variant in ("cfr+", "dcfr"):
        nplayer.test_one_iteration_parity(name, variant, precision, tol)


@pytest.mark.parametrize("precision,tol", [("f32", 1e-6), ("f64", 1e-12)])
def test_general_sum_bench_game_launches(monkeypatch, precision, tol):
    """And of four wavefronts."""
    import bench
    monkeypatch.setattr(nplayer, "_solver", _by_level_n)
    nplayer.test_bench_game_one_iteration_full_size(games.random_game_n(**bench.NPLAYER_GAME),
                                                    precision, tol)


def test_general_sum_graph_replay():
    """More actions than the one launch takes: a captured graph of the level kernels."""
    from paper_2408_14778_amd import NPlayerSolver
    rng = np.random.default_rng(3)
    g = games.normal_form_n(rng.integers(-64, 65, size=(17, 3, 4, 3)) / 64.0, name="nf17")
    a, b = (NPlayerSolver(g, "cfr+", graph=graph) for graph in (True, False))
    assert not a.one_launch
    for s in (a, b):
        s.iterate(7)
    for x, y in zip(a.get_state(), b.get_state()):
        assert np.array_equal(x, y)


# a hidden width, an input width and a slot count that the fused step does not take
@pytest.mark.parametrize("F,H,A,rows", [(96, 192, 4, 63), (88, 256, 4, 300), (96, 128, 12, 545)])
def test_training_step_layer_by_layer(F, H, A, rows):
    fused.test_training_step(F, H, A, rows)
