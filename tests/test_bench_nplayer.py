"""bench.py's three-player line keeps the two routes apart: a level-by-level kernel's time is a share of
level-by-level iterations, whatever the solver's own route takes."""
import argparse

import numpy as np
import pytest

import bench
import games
import paper_2408_14778_amd as pkg
from oracle.layout import canonical_layout

ONE_S, LEVEL_S = 80e-6, 150e-6


def _fake(game, resident):
    lay = canonical_layout(game)

    class Fake:
        made = []

        def __init__(self, g, variant, precision, schedule, graph=True):
            self.n_q, self.one_launch = 3, resident and graph
            Fake.made.append(graph)

        def iterate(self, n):
            pass

        def iterate_timed(self, n):
            # only a solver that runs level by level may give the level kernels' times
            assert not self.one_launch
            return {"value_level": (8 * n, 0.1 * n), "reach_level": (9 * n, 0.05 * n)}

        def layout(self, name):
            if name == "one_launch":
                return np.array([1, 256, 400, 100] if self.one_launch else [0] * 4, dtype=np.int32)
            return lay[name]

        def close(self):
            pass

    return Fake


@pytest.mark.parametrize("resident", [True, False])
def test_kernel_shares_are_of_the_route_they_ran_on(monkeypatch, resident):
    g = games.normal_form_n(np.arange(36.0).reshape(2, 3, 2, 3) / 64)
    fake = _fake(g, resident)
    monkeypatch.setattr(pkg, "NPlayerSolver", fake)
    monkeypatch.setattr(bench, "_timed", lambda s, steps: (ONE_S, ONE_S) if s.one_launch
                        else (LEVEL_S, LEVEL_S))
    args = argparse.Namespace(precision="f32", schedule="simultaneous", warmup=1, steps=10,
                              timed_kernel_steps=4)
    out = bench.bench_nplayer(args, g)
    assert fake.made == ([True, False] if resident else [True])
    own = ONE_S if resident else LEVEL_S
    assert out["ms_per_step"] == own * 1e3 and out["value"] == g.n_nodes / own
    r = out["roofline"]
    assert r["kernel"] == "value_level"
    assert np.isclose(r["avg_launch_us"], LEVEL_S * 1e6 * (0.1 / 0.15) / 8)
    assert r["iteration_us_events"] == LEVEL_S * 1e6
    assert ("node engine" in out["config"]["workload"]) != resident
    assert (out["one_launch"] is not None) == resident
