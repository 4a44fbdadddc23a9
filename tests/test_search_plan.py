"""The room a search is given in its workspace (csrc/search_plan.h): enough for the tiles that calls make, and never less
for a call of more queries or probes, because a recorded graph stays valid only while no later, smaller call moves a buffer.

Score rows and per-query arrays are checked the same way at workspace limits that cut calls into passes (there a call
with shorter rows has longer passes, and one with as many bytes may round to more or fewer rows).

The exact redo's launches are checked to find a score row for every query that they share out at a time, and enough queries or
workgroups a query to have work for at least half of the workgroups.

Tiles are dealt out to queues: every tile to one, and every queue has a workgroup, on a chip that holds fewer workgroups than queues too.

The grid holds the calls at which cutting lists more finely for fewer pairs would need more tiles than the larger call has
(10M vectors, 32 probes: 387 | 388 queries over 4000 lists, 195 | 196 over 2000) and an index with one hot list."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_room_never_falls_and_holds_every_call(tmp_path):
    exe = str(tmp_path / "search_plan")
    build = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2605_17415_amd", "csrc"),
                            os.path.join(ROOT, "tests", "search_plan_driver.cpp"), "-o", exe], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0 and run.stdout == "ok\n", run.stdout + run.stderr
