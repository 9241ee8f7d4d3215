"""The default number of shares of a batched class (batch_plan.h), on the CPU:
within its limits and covering every cube once at the edges of its range."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2302_05730_amd", "csrc")

SOURCE = r"""
#include <stdio.h>
#include <stdlib.h>
#include "batch_plan.h"
using namespace mcubes;
// items, cubes of each, samples per cube, dimension, block, resident, CUs, bins -> shares, tiles
int main(int, char **v) {
    const int64_t n = atoll(v[1]), m = atoll(v[2]), p = atoll(v[3]);
    const int dim = atoi(v[4]), block = atoi(v[5]), resident = atoi(v[6]), cus = atoi(v[7]);
    const int most = class_shares(n * m, block, resident, 0, 8, 1 << 20);
    const int64_t shares =
        default_shares(dim, n, n * m, n * m * p, atoi(v[8]) != 0, block, resident, cus, most);
    if (shares < 1 || shares > most) return 1;
    std::vector<int> items;
    for (int i = 0; i < n; ++i) items.push_back(i);
    const std::vector<int64_t> ms(n, m), ps(n, p);
    std::vector<BatchTile> tiles;
    split_tiles(items, ms.data(), ps.data(), (int)shares, tiles);
    int64_t covered = 0;
    for (const BatchTile &t : tiles) covered += (int64_t)t.w_end - t.w_begin;
    if (covered != n * m) return 2;
    printf("%lld %zu\n", (long long)shares, tiles.size());
    return 0;
}
"""


@pytest.fixture(scope="module")
def split(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("split")
    (d / "split.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", f"-I{CSRC}", str(d / "split.cpp"), "-o",
                    str(d / "split")], check=True, timeout=120)

    def run(*args):
        out = subprocess.run([str(d / "split"), *map(str, args)], check=True, timeout=60,
                             capture_output=True, text=True).stdout
        return tuple(map(int, out.split()))
    return run


@pytest.mark.parametrize("case", [
    (1, 1, 2, 2, 512, 1024, 256, 1),            # one cube
    (1, 1, 5_000_000, 8, 512, 256, 256, 1),     # one cube of all the samples
    (1, 513, 2, 3, 512, 1024, 256, 1),          # one cube more than a workgroup
    (7, 100_003, 2, 4, 512, 1024, 256, 0),      # no bin sums
    (3, 65_536, 11, 8, 64, 1, 1, 1),            # one slot
    (1, 4_294_967_295, 2, 8, 512, 512, 256, 1),  # the largest integrand
    (3000, 3, 2, 5, 512, 1024, 256, 1),         # more integrands than slots
])
def test_default_split_in_range(split, case):
    split(*case)


def test_small_class_in_one_round(split):
    """Four cubes per thread of every slot: no more workgroups than slots."""
    assert split(1, 2_000_000, 2, 2, 512, 1024, 256, 1)[1] <= 1024
