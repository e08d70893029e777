"""The out-of-core stream's plan and the batch joined under one root, decoded and compared with the
canonical layouts record by record on the host, under the address and undefined-behaviour sanitizers."""
import os
import shutil
import subprocess

import pytest

import games
from test_gpu_partitioned_stream import _uneven
from test_host_sanitized import CSRC, ROOT, _write


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_stream_and_forest_plans(tmp_path):
    exe = str(tmp_path / "stream_driver")
    src = [os.path.join(CSRC, f) for f in ("flatten.cpp", "partition_plan.cpp", "stream_plan.cpp",
                                           "resident_plan.cpp")]
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-pthread", *src,
                    os.path.join(ROOT, "tests", "host_check", "stream_driver.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    data = str(tmp_path / "games.bin")
    _write(data, [games.kuhn_like(3, "joint"), games.kuhn_like(3, "sequential").permuted(2),
                  games.leduc_like(3, 2, deal="sequential"), games.rock_paper_scissors(),
                  games.random_game(22, deal="sequential", depth=6), _uneven(),
                  games.random_game(66, deal="sequential", depth=30, max_actions=2, p_terminal=0.3),
                  games.random_game(72, deal="joint", depth=3, max_actions=16),
                  games.poker_game(7, 2, 2, 60, max_deals=5)])
    r = subprocess.run([exe, data], capture_output=True, text=True, timeout=600)
    print(r.stdout[-2000:])
    assert r.returncode == 0, r.stdout[-500:] + r.stderr[-4000:]
    assert r.stdout.strip().endswith("ok")
