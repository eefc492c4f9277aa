"""The limits that the host keeps when it chooses a schedule
(csrc/qc_schedule.h), built on their own by the host compiler and checked by
tests/schedule_driver.cpp; and that the calls which hold spare memory go through
them.  CPU only."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2412_10072_amd", "csrc")


def test_limits(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    exe = str(tmp_path / "schedule")
    cmd = [cxx, "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-Wall", "-Werror",
           os.path.join(HERE, "schedule_driver.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, f"build failed:\n{res.stdout}\n{res.stderr}"
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "0 failures" in run.stdout, f"{run.stdout}\n{run.stderr}"


def test_spare_buffers_grow_within_the_limits():
    """The folded model, the phasor table and the outputs' table are taken by
    spare_memory, never grown outright."""
    text = open(os.path.join(CSRC, "qc_api.hip")).read()
    for buf in ("d_fold", "d_ptab", "d_outtab"):
        assert re.search(r"spare_memory\(ctx, ctx->%s\b" % buf, text), buf
        assert not re.search(r"grow\(ctx->%s\b" % buf, text), buf


def test_batch_teams_give_way_to_the_buckets():
    """The teams' memory is asked for within the limits, and a batch without it goes
    to the buckets instead of failing."""
    text = open(os.path.join(CSRC, "qc_batch_api.hip")).read()
    make = text[text.index("qc_status make_team("):]
    make = make[:make.index("\n}\n")]
    assert make.index("spare_fits(") < make.index("hipMalloc(")
    create = text[text.index("qc_status qc_batch_create("):]
    assert re.search(r"st = make_team\(b, sorted\);\s+if \(st == QC_E_NOMEM\) \{[^}]*arrange\(b, items, team, sorted\);"
                     r"\s+st = QC_OK;", create)
