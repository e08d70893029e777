"""The resident iteration's plan, followed record by record on the host and compared with the canonical
layouts, and without memory: under the address and undefined-behaviour sanitizers."""
import os
import re
import shutil
import subprocess

import pytest

import games
from test_host_sanitized import CSRC, ROOT, _write

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("resident") / "resident_driver")
    src = [os.path.join(CSRC, f) for f in ("flatten.cpp", "resident_plan.cpp")]
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-pthread", *src,
                    os.path.join(ROOT, "tests", "host_check", "resident_driver.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    return exe


def _run(driver, path, *args):
    r = subprocess.run([driver, path, *args], capture_output=True, text=True, timeout=600)
    print(r.stdout[-2000:])
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    assert r.stdout.strip().endswith("ok")
    return r.stdout


def test_records(driver, tmp_path):
    data = str(tmp_path / "games.bin")
    _write(data, [games.kuhn_like(3, "joint"), games.kuhn_like(35, "joint"),
                  games.kuhn_like(3, "sequential").permuted(2),
                  games.leduc_like(3, 2, deal="sequential"), games.leduc_like(6, 2, deal="joint"),
                  games.rock_paper_scissors(), games.random_game(22, deal="sequential", depth=6),
                  games.random_game(66, deal="sequential", depth=30, max_actions=2, p_terminal=0.3),
                  games.random_game(72, deal="joint", depth=3, max_actions=16),
                  games.poker_game(7, 2, 2, 60, max_deals=5), games.poker_game(10, 3, 1, 60, max_deals=31),
                  games.kuhn3(), games.random_game_n(3, 3, 9, 5), games.random_game_n(6, 3, 12, 5),
                  games.random_game_n(3, 8, 2, 4), games.leduc_like(4, 2, deal="sequential")])
    out = _run(driver, data)
    solo, team = map(int, re.search(r"(\d+) of one workgroup, (\d+) of teams", out).groups())
    assert solo >= 10 and team >= 10


def test_no_memory(driver, tmp_path):
    data = str(tmp_path / "games.bin")
    _write(data, [games.kuhn_like(3, "joint"), games.leduc_like(4, 2, deal="sequential"),
                  games.random_game_n(3, 3, 7, 5)])
    _run(driver, data, "starve")
