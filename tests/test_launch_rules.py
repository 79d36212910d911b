"""Host-side launch rules of the 2D passes (csrc/launch_rules.hpp), compiled into
a small program.  Runs on the CPU."""
import os
import subprocess

import pytest

from paper_1402_5670_amd import build as bld

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "launch_rules_model")
    subprocess.run([bld.hipcc(), *bld.COMMON, "-x", "hip", "-I", bld.CSRC,
                    os.path.join(HERE, "launch_rules_model.cpp"), "-o", exe],
                   check=True, capture_output=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=60).stdout
    lines = {}
    for w in (line.split() for line in out.splitlines()):
        lines.setdefault(w[0], []).append([int(v) for v in w[1:]])
    return lines


def test_few_rows_are_fewer_rows(rules):
    # the blocks for small grids hold at most the lines of the ordinary ones
    assert len(rules["rows"]) == 15
    for n, tile, few in rules["rows"]:
        assert 1 <= few <= tile, n
        assert n < 256 or few <= tile // 4, n


def test_failed_occupancy_query_leaves_no_error(rules):
    # one block per compute unit, and no error left for the check after the next
    # launch
    assert rules["resident"] == [[256, 0]]
