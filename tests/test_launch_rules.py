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


def test_forward_split(rules):
    # 256 compute units of 4 resident blocks, 9 pairs; the cost of a split is its
    # rounds times the pairs of a part.  256 blocks: 3 parts (1 round of 3, for 9
    # whole and 1 x 5 in two); 384: 5 parts (2 x 2, for 1 x 5 in two); 512 and 1024
    # blocks are resident at once, two or four per unit, and left whole; 1030 take
    # 3 parts (4 x 3, for 2 x 9 whole)
    assert dict(rules["forward"]) == {256: 3, 384: 5, 512: 1, 1024: 1, 1030: 3}
