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
int main(int argc, char** argv)  // B * H, rows, bytes of a row
{
    for (int i = 1; i + 2 < argc; i += 3) {
        const int BH = atoi(argv[i]);
        printf("%d %d\n", ec::decode_auto_splits(BH, atoi(argv[i + 1]), atoi(argv[i + 2])), ec::split_stride(BH));
    }
}
"""


@pytest.fixture(scope="module")
def divided(tmp_path_factory):
    """(shares of a pair, workgroups per share) of calls (B * H, rows, bytes of a row)."""
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
        for BH, (splits, stride) in zip(pairs, divided([(BH, rows, 256) for BH in pairs])):
            assert stride % 8 == 0 and BH <= stride < BH + 8
            assert splits == 1 or stride // 8 * splits <= 32, (BH, rows, splits)


def test_long_caches_are_divided_as_far_as_an_xcd_has_room(divided):
    calls = [(8, 8192, 256), (16, 8192, 256), (8, 2000, 256), (24, 8192, 256), (32, 640, 256), (33, 8192, 256), (48, 8192, 256),
             (64, 8192, 256), (80, 8192, 256), (96, 8192, 256), (128, 8192, 256), (129, 8192, 256)]
    assert [s for s, _ in divided(calls)] == [16, 16, 8, 8, 8, 6, 5, 4, 3, 2, 2, 1]


def test_workgroups_exchange_at_device_scope():
    """Words that pass between workgroups are no business of a workgroup alone: a compiler may drop or merge accesses of that scope."""
    for path in glob.glob(os.path.join(CSRC, "*")):
        text = open(path).read()
        assert "HIP_MEMORY_SCOPE_WORKGROUP" not in text and "HIP_MEMORY_SCOPE_WAVEFRONT" not in text, path
