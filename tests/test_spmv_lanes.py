"""The lanes per block row that a handle's SpMV takes without being tuned (spmv_lanes in
dpcg_internal.h), against measured times, on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# block rows, mean and longest row in blocks, us of the iteration's SpMV with 4, 8, 16 and 32
# lanes per row (one MI355X): bands, bands with six long rows, and half the rows in a band
MEASURED = [
    (1500, 5.0, 5, (5.61, 5.43, 5.66, 5.57)),
    (1500, 11.0, 11, (6.09, 5.60, 5.27, 5.37)),
    (1500, 20.9, 21, (7.45, 6.23, 6.01, 5.65)),
    (1500, 5.5, 69, (11.07, 8.52, 6.53, 5.92)),
    (1500, 8.2, 405, (34.37, 19.84, 12.51, 8.83)),
    (1500, 14.0, 141, (17.12, 11.15, 7.83, 6.41)),
    (1500, 6.0, 11, (5.85, 5.60, 5.29, 5.22)),
    (20000, 3.0, 3, (5.72, 5.92, 6.62, 8.73)),
    (20000, 7.0, 7, (6.73, 6.41, 7.25, 8.95)),
    (20000, 13.0, 13, (8.65, 6.92, 7.05, 9.00)),
    (20000, 21.0, 21, (12.94, 10.03, 8.83, 9.11)),
    (20000, 27.0, 27, (16.90, 12.59, 10.74, 10.31)),
    (20000, 5.0, 37, (8.54, 7.03, 7.85, 8.68)),
    (20000, 5.1, 133, (16.60, 11.47, 9.14, 8.86)),
    (20000, 5.2, 405, (38.98, 23.13, 15.51, 12.47)),
    (20000, 13.2, 413, (40.00, 23.89, 18.68, 13.15)),
    (20000, 6.0, 11, (6.48, 5.91, 6.88, 8.43)),
    (200000, 3.0, 3, (11.52, 14.92, 24.08, 43.37)),
    (200000, 5.0, 5, (18.01, 15.84, 24.19, 43.53)),
    (200000, 9.0, 9, (30.26, 25.41, 25.35, 44.52)),
    (200000, 13.0, 13, (65.20, 33.20, 31.07, 47.51)),
    (200000, 23.0, 23, (207.68, 86.01, 75.66, 76.73)),
    (200000, 33.0, 33, (311.50, 139.99, 113.46, 122.06)),
    (200000, 5.0, 69, (22.24, 18.05, 24.95, 43.45)),
    (200000, 5.0, 405, (56.12, 36.01, 33.24, 45.78)),
    (200000, 13.0, 413, (99.31, 49.47, 39.69, 48.08)),
    (200000, 6.0, 11, (25.24, 21.79, 25.44, 43.58)),
]

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>

#include "dpcg_internal.h"

int main(int argc, char **argv) {
    for (int i = 1; i + 2 < argc; i += 3)
        printf("%d\n", dpcg::spmv_lanes(atoi(argv[i]), atoll(argv[i + 1]), atoi(argv[i + 2])));
    return 0;
}
"""


@pytest.fixture(scope="module")
def lanes(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("lanes")
    src, exe = d / "lanes.cpp", str(d / "lanes")
    src.write_text(PROGRAM)
    subprocess.check_call([HIPCC, "-O1", "-std=c++17", "-x", "hip", "--offload-host-only", "-I",
                           os.path.join(ROOT, "paper_2111_09294_amd", "csrc"), str(src), "-o", exe])

    def run(cases):
        args = [str(int(v)) for c in cases for v in c]
        return [int(v) for v in subprocess.check_output([exe] + args, text=True).split()]

    return run


def test_choice_is_near_the_fastest(lanes):
    got = lanes([(nb, round(mean * nb), longest) for nb, mean, longest, _ in MEASURED])
    for g, (nb, mean, longest, us) in zip(got, MEASURED):
        assert us[(4, 8, 16, 32).index(g)] <= 1.1 * min(us), (nb, mean, longest, g)


def test_edges(lanes):
    """No rows, one block per row, the lines of the mean, the longest possible row."""
    big = 10 ** 7  # enough rows that the launch outweighs any chain of these lengths
    cases = [(0, 0, 0), (1, 1, 1), (big, 4 * big, 4), (big, 4 * big + 1, 5), (big, 10 * big, 10),
             (big, 10 * big + 1, 11), (big, 22 * big, 22), (big, 22 * big + 1, 0), (5, 25, 5), (2 ** 29, 2 ** 30, 2 ** 29)]
    assert lanes(cases) == [4, 4, 4, 8, 8, 16, 16, 32, 8, 32]
