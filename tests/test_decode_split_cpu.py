"""How a generation step is divided over workgroups, looked at without a GPU."""
import glob
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_18121_amd", "csrc")

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include "decode_split.h"
int main(int argc, char** argv)  // B * H, rows, bytes of a row, bf16; or "lines", shares of a pair, number of the first output row, pairs
{
    if (argc > 4 && argv[1][0] == 'l') {
        for (int bh = 0; bh < atoi(argv[4]); ++bh) printf("%d %u\n", bh % ec::kXcds, ec::first_line(atoll(argv[3]) + bh, atoi(argv[2])));
        return 0;
    }
    for (int i = 1; i + 3 < argc; i += 4) {
        const int BH = atoi(argv[i]);
        printf("%d %d\n", ec::decode_auto_splits(BH, atoi(argv[i + 1]), atoi(argv[i + 2]), atoi(argv[i + 3])), ec::split_stride(BH));
    }
}
"""


@pytest.fixture(scope="module")
def divided(tmp_path_factory):
    """(shares of a pair, workgroups per share) of calls (B * H, rows, bytes of a row, bf16)."""
    at = tmp_path_factory.mktemp("split")
    source, binary = at / "split.cpp", at / "split"
    source.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", str(binary), str(source)], check=True)

    def run(calls):
        args = [str(x) for c in calls for x in c]
        lines = subprocess.run([str(binary), *args], check=True, capture_output=True, text=True).stdout.splitlines()
        return [tuple(int(x) for x in line.split()) for line in lines]
    return run


def test_no_xcd_gets_more_workgroups_than_it_has_compute_units(divided):
    """A pair's workgroups are on one XCD: its pairs, the most that any of the eight has, share 32 compute units."""
    for rows in (300, 640, 1030, 3100, 4400, 100000):
        pairs = range(1, 400)
        for BH, (splits, stride) in zip(pairs, divided([(BH, rows, 256, 1) for BH in pairs])):
            assert stride % 8 == 0 and BH <= stride < BH + 8
            assert splits == 1 or stride // 8 * splits <= 32, (BH, rows, splits)


def test_long_caches_are_divided_as_far_as_an_xcd_has_room(divided):
    calls = [(8, 8192), (16, 8192), (8, 2000), (24, 8192), (32, 640), (33, 8192), (48, 8192), (64, 8192), (80, 8192), (96, 8192), (128, 8192), (129, 8192)]
    assert [s for s, _ in divided([(*c, 256, 1) for c in calls])] == [16, 16, 8, 8, 8, 6, 5, 4, 3, 2, 2, 1]


def test_short_caches_are_left_alone(divided):
    """On both sides of the size from which dividing a pair is measured to be faster (KB of K and V)."""
    bf16_d128 = ((1, 256, 8), (40, 268, 6), (48, 292, 5), (49, 320, 4), (64, 340, 4), (65, 343, 3), (80, 388, 3), (81, 423, 2), (96, 468, 2), (97, 960, 2))
    others = ((1, 240, 8), (40, 252, 6), (48, 276, 5), (49, 320, 4), (64, 324, 4), (65, 327, 3), (80, 372, 3), (81, 407, 2), (96, 452, 2), (97, 960, 2))
    for row, half, table in ((256, 1, bf16_d128), (256, 0, others), (512, 0, others), (128, 1, others)):
        for BH, kb, shares in table:
            rows = kb * 512 // row
            assert [s for s, _ in divided([(BH, rows - 1, row, half), (BH, rows, row, half)])] == [1, shares]


def test_pairs_that_meet_on_an_xcd_have_lines_of_their_own(divided):
    """As long as 256 lines are enough for the shares of an XCD's pairs, wherever the output lies."""
    for splits in (2, 3, 8, 9, 16, 17, 32, 33, 64):
        pairs = 8 * (256 // (splits - 1))
        for row in (0, 5, 123456789, (1 << 47) // 256):
            lines = {}
            for xcd, first in divided([("lines", splits, row, pairs)]):
                lines.setdefault(xcd, []).extend((first + s) % 256 for s in range(splits - 1))
            assert len(lines) == 8
            for used in lines.values():
                assert len(set(used)) == len(used) <= 256, (splits, row)


def test_workgroups_exchange_at_device_scope():
    """Words that pass between workgroups are no business of a workgroup alone: a compiler may drop or merge accesses of that scope."""
    for path in glob.glob(os.path.join(CSRC, "*")):
        text = open(path).read()
        assert "HIP_MEMORY_SCOPE_WORKGROUP" not in text and "HIP_MEMORY_SCOPE_WAVEFRONT" not in text, path
