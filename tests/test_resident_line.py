"""Which games are planned to iterate in one launch, by the workspace that cfr_plan reports (no GPU):
the same game asked to run level by level has none of its records."""
import ctypes

import games


def _bytes(g, **kw):
    from paper_2408_14778_amd import _native as N
    from paper_2408_14778_amd.solver import GameArgs, make_config
    args, cfg, info = GameArgs(g), make_config("cfr+", **kw), N.CfrPlanInfo()
    N.check(N.load().cfr_plan(ctypes.byref(args.struct), ctypes.byref(cfg), ctypes.byref(info)))
    return int(info.workspace_bytes)


def _one_launch(g, **kw):
    return _bytes(g, **kw) > _bytes(g, graph=False, **kw)


def test_line_of_single_precision_games():
    """Past 6.4 million nodes the public-block launches are faster, of two passes past 7 million."""
    small = games.poker_game(13, 3, 3, 400, max_deals=46)
    assert small.n_nodes == 6342481
    assert _one_launch(small) and _one_launch(small, schedule="alternating")
    large = games.poker_game(12, 3, 2, 300, max_deals=110)
    assert large.n_nodes == 6596371
    assert not _one_launch(large)
    assert _one_launch(large, schedule="alternating") and _one_launch(large, precision="f64")


def test_no_workspace_for_records_that_cannot_fit(large_game):
    """21.5 million nodes in double precision: three times what eight bins per workgroup hold."""
    assert not _one_launch(large_game, precision="f64")
    assert not _one_launch(large_game) and not _one_launch(large_game, schedule="alternating")
