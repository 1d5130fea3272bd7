"""The rule that sends a scoring call to its kernels, compiled by itself: a head has to fit into the 32-bit byte offsets
of the matrix-core kernels' buffer descriptors, whatever else is true of the call.  No kernels run."""
import os
import subprocess

import pytest

from paper_2407_18121_amd import binding as ec

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_18121_amd", "csrc")
MFMA, F32, SIMT, MFMA_OFF_GRID = range(4)
PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include "score_route.h"
int main(int argc, char** argv)
{
    if (argc > 1 && argv[1][0] == 'p') {  // pairs: D, tiles, heads, Tq, P
        for (int i = 2; i + 4 < argc; i += 5) {
            long long a[5];
            for (int j = 0; j < 5; ++j) a[j] = atoll(argv[i + j]);
            printf("%d\n", ec::pair_query_tiles((int)a[0], a[1], a[2], a[3], a[4]) + 2 * ec::pair_key_tiles((int)a[0], a[1], a[2], a[3], a[4]));
        }
        return 0;
    }
    for (int i = 1; i + 6 < argc; i += 7) {
        const char* base = (const char*)(uintptr_t)(1 << 20);  // only the low bits of the addresses matter
        const void* p[4];
        for (int j = 0; j < 4; ++j) p[j] = base + atoi(argv[i + 3 + j]);
        printf("%d\n", (int)ec::score_route(atoi(argv[i]), atoi(argv[i + 1]), atoll(argv[i + 2]), p[0], p[1], p[2], p[3]));
    }
}
"""


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    at = tmp_path_factory.mktemp("route")
    source, binary = at / "route.cpp", at / "route"
    source.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", str(binary), str(source)], check=True)

    def run(calls, pairs=False):
        if pairs:
            args = ["p"] + [str(x) for c in calls for x in c]
            return [(int(x) & 1, int(x) >> 1) for x in subprocess.run([str(binary), *args], check=True, capture_output=True, text=True).stdout.split()]
        args = [str(x) for dt, D, rows, offsets in calls for x in (dt, D, rows, *offsets)]
        return [int(x) for x in subprocess.run([str(binary), *args], check=True, capture_output=True, text=True).stdout.split()]
    return run


ON = (0, 0, 0, 0)


@pytest.mark.parametrize("dt,D,matrix", [(ec.EC_F32, 128, F32), (ec.EC_F32, 64, F32), (ec.EC_BF16, 128, MFMA), (ec.EC_BF16, 64, MFMA)])
def test_heads_beyond_the_descriptors_take_the_vector_kernels(route, dt, D, matrix):
    row = D * (4 if dt == ec.EC_F32 else 2)
    most = 2 ** 32 // row  # rows of 4 GiB
    got = route([(dt, D, rows, ON) for rows in (1, 2 ** 31 // row, most - 1024, most - 1023, most, most + 1, 2 ** 30)])
    assert got == [matrix] * 3 + [SIMT] * 4


def test_rows_off_the_16_byte_grid(route):
    """bf16 stays on the matrix cores wherever its tensors start; out may start anywhere in either of its forms."""
    for off in ((2, 0, 0, 0), (0, 2, 0, 0), (0, 0, 8, 0), (2, 4, 8, 6)):
        assert route([(ec.EC_BF16, D, rows, off) for D in (64, 128) for rows in (1, 500, 100000)]) == [MFMA_OFF_GRID] * 6
    assert route([(ec.EC_BF16, 64, 500, off) for off in (ON, (0, 0, 0, 2), (16, 32, 48, 64))]) == [MFMA] * 3
    assert route([(ec.EC_F32, 64, 500, off) for off in (ON, (16, 32, 48, 64))]) == [F32] * 2
    assert route([(ec.EC_F32, 64, 500, tuple(4 * (j == i) for j in range(4))) for i in range(4)]) == [SIMT] * 4


def test_pairs_of_tiles(route):
    """(query tiles in pairs, key tiles in pairs) on either side of every bound of the two rules."""
    cases = [  # D, tiles, heads, Tq, P -> query, key
        ((128, 3, 4096, 384, 0), (0, 0)), ((128, 4, 128, 512, 0), (1, 1)), ((128, 4, 127, 512, 0), (0, 0)),   # tiles, one per unit
        ((128, 4, 128, 512, 256), (1, 1)), ((128, 4, 128, 512, 257), (1, 0)), ((128, 4, 128, 512, 513), (0, 0)),  # prefix
        ((128, 8, 64, 1024, 0), (1, 1)), ((128, 8, 65, 1024, 0), (1, 0)), ((128, 8, 95, 1024, 0), (1, 0)),     # 256, 260, 380
        ((128, 8, 96, 1024, 0), (1, 1)), ((128, 8, 132, 1024, 0), (1, 1)), ((128, 8, 133, 1024, 0), (0, 1)),   # 384, 528, 532
        ((128, 8, 153, 1024, 0), (0, 1)), ((128, 8, 154, 1024, 0), (1, 1)),                                    # 612, 616 of 1024
        ((128, 11, 171, 1400, 0), (0, 1)), ((128, 13, 146, 1600, 0), (1, 1)), ((128, 5, 64, 640, 0), (0, 0)),  # odd tiles
        ((64, 8, 64, 1024, 0), (1, 1)), ((64, 8, 75, 1024, 0), (0, 0)), ((64, 8, 76, 1024, 0), (1, 0)),         # 256, 300, 304
        ((64, 6, 128, 768, 0), (0, 1)), ((64, 6, 160, 768, 0), (1, 1)), ((64, 4, 239, 512, 0), (0, 1)), ((64, 4, 240, 512, 0), (1, 1)),
        ((64, 8, 179, 1024, 0), (0, 0)), ((64, 8, 180, 1024, 0), (1, 1)),                                      # 716, 720 of 1024
        ((64, 13, 136, 1600, 0), (0, 1)), ((64, 13, 137, 1600, 0), (1, 1)), ((64, 11, 256, 1400, 0), (0, 1)),   # odd: 952, 959; 11 tiles
    ]
    assert route([c for c, _ in cases], pairs=True) == [x for _, x in cases]
