"""The tuner's cache file (GPU): an entry of the present kernels is taken, one whose key carries no
version, as keys once did, is measured anew."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PLAN = ("import paper_2510_27351_amd as wf\n"
        "p = wf.Plan([300, 64, 200], [100, 257, 65])\n"
        "print(p.tile, p.rows)\n")


def make_plan(cache):
    # a process of its own: the file is read once per process
    out = subprocess.run([sys.executable, "-c", PLAN], cwd=ROOT, env={**os.environ, "WF_TUNE_CACHE": str(cache)},
                         check=True, stdout=subprocess.PIPE, text=True, timeout=100).stdout
    return out.split()[-2:]


def test_entries_of_other_versions_are_not_taken(tmp_path):
    cache = tmp_path / "tune.txt"
    config = make_plan(cache)
    (key, *found), = [line.split() for line in cache.read_text().splitlines()]
    assert found == config
    version, _, rest = key.partition("-")
    assert version[0] == "v" and version[1:].isdigit()
    # a configuration that the tuner did not choose shows where it came from
    other = ["64" if config[0] != "64" else "16", "1" if config[1] != "1" else "2"]
    cache.write_text(" ".join([key, *other]) + "\n")
    assert make_plan(cache) == other
    assert len(cache.read_text().splitlines()) == 1
    cache.write_text(" ".join([rest, *other]) + "\n")
    make_plan(cache)
    lines = [line.split() for line in cache.read_text().splitlines()]
    assert lines[0] == [rest, *other] and [line[0] for line in lines[1:]] == [key]
