"""The default split of a batched class (batch_plan.h), on the CPU: classes of thousands of integrands
with a large one among them, and classes of much work."""
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
// small integrands and their cubes, large integrands and theirs, samples per cube, dimension, block,
// resident, CUs -> shares, tiles, cubes of the class, cubes of the largest tile
int main(int, char **v) {
    const int64_t small = atoll(v[1]), m0 = atoll(v[2]), large = atoll(v[3]), m1 = atoll(v[4]);
    const int64_t p = atoll(v[5]), n = small + large;
    const int dim = atoi(v[6]), block = atoi(v[7]), resident = atoi(v[8]), cus = atoi(v[9]);
    std::vector<int> items;
    std::vector<int64_t> ms, ps(n, p);
    int64_t cubes = 0;
    for (int i = 0; i < n; ++i) {
        items.push_back(i);
        ms.push_back(i < small ? m0 : m1);
        cubes += ms.back();
    }
    const int most = class_shares(cubes, block, resident, 0, 8, 1 << 20);
    const int64_t shares =
        default_shares(dim, n, cubes, cubes * p, true, block, resident, cus, most);
    if (shares < 1 || shares > most) return 1;
    std::vector<BatchTile> tiles;
    split_tiles(items, ms.data(), ps.data(), (int)shares, tiles);
    int64_t covered = 0, largest = 0;
    for (const BatchTile &t : tiles) {
        covered += (int64_t)t.w_end - t.w_begin;
        largest = std::max(largest, (int64_t)t.w_end - t.w_begin);
    }
    if (covered != cubes) return 2;
    printf("%lld %zu %lld %lld\n", (long long)shares, tiles.size(), (long long)cubes, (long long)largest);
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


@pytest.mark.parametrize("small", [0, 1, 500, 2500, 4095, 4096, 4097, 6000, 60000])
@pytest.mark.parametrize("dim", [2, 3, 8])
def test_a_large_integrand_is_cut_whatever_its_company(split, small, dim):
    """One integrand of 5e7 cubes among many of 343: no workgroup takes more than the 256 CUs' share of
    it twice over."""
    _, _, cubes, largest = split(small, 343, 1, 50_000_000, 2, dim, 512, 512, 256)
    assert largest <= 2 * cubes / 256


@pytest.mark.parametrize("items", [1, 8, 64])
@pytest.mark.parametrize("dim,m", [(2, 125_000_000), (3, 125_000_000), (5, 100_000_000), (8, 43_046_721)])
def test_a_large_class_fills_several_rounds(split, items, dim, m):
    """2.5e8 samples of one family and more: two rounds at least (eight of 5e7 samples took 2 to 7% more
    in one), and no tile twice its share."""
    shares, tiles, cubes, largest = split(0, 1, items, m // items, 2, dim, 512, 512, 256)
    assert tiles >= 2 * 512 and largest <= 2 * cubes / shares


@pytest.mark.parametrize("items", [1, 8])
@pytest.mark.parametrize("dim,m", [(2, 500_000), (3, 500_000), (5, 500_000), (8, 390_625)])
def test_a_small_class_stays_in_one_round(split, items, dim, m):
    """1e6 samples in all: every workgroup's tables and histogram cost more than its samples."""
    assert split(0, 1, items, m // items, 2, dim, 512, 512, 256)[1] <= 512
