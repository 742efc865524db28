"""How the causal pass deals its items to the dies (CPU only): the header's own functions, compiled for the host."""
import shutil
import subprocess

import pytest

from paper_2508_11553_amd import build as sd_build
from tests.test_kernel_resources import CSRC

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "kernels.h"
int main(int argc, char **argv)
{
    const int q_blocks = atoi(argv[1]), pairs = atoi(argv[2]);
    const unsigned grid = sd::prefill_grid(q_blocks, pairs);
    std::vector<int> seen((size_t)pairs * q_blocks, 0), per_die(sd::kXcds, 0);
    for (unsigned i = 0; i < grid; ++i) {
        const sd::PrefillItem it = sd::prefill_item(i, q_blocks, pairs);
        if (it.pair < 0 || it.pair >= pairs || it.block < 0) return 2;
        if (it.block >= q_blocks) continue;
        seen[(size_t)it.pair * q_blocks + it.block]++;
        per_die[i % sd::kXcds]++;
    }
    int missing = 0, lo = per_die[0], hi = per_die[0];
    for (int s : seen) missing += s != 1;
    for (int n : per_die) lo = n < lo ? n : lo, hi = n > hi ? n : hi;
    printf("%u %d %d %d\n", grid, missing, lo, hi);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which(sd_build.HIPCC) is None:
        pytest.skip("needs hipcc")
    d = tmp_path_factory.mktemp("geometry")
    (d / "items.hip").write_text(PROGRAM)
    r = subprocess.run([sd_build.HIPCC, "--offload-host-only", "-std=c++17", f"-I{CSRC}", str(d / "items.hip"), "-o", str(d / "items")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return str(d / "items")


@pytest.mark.parametrize("pairs", [1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 20, 28, 64, 96, 1023])
@pytest.mark.parametrize("q_blocks", [1, 2, 7, 8, 9, 64, 129])
def test_every_item_is_dealt_once_and_to_every_die_alike(program, q_blocks, pairs):
    grid, missing, lo, hi = map(int, subprocess.run([program, str(q_blocks), str(pairs)], capture_output=True, text=True, check=True).stdout.split())
    assert missing == 0
    assert grid % 8 == 0 and grid < pairs * q_blocks + 7 * 8   # what is padded: a class's last block of a left-over pair
    assert hi - lo <= 7   # at most one block per left-over pair
