"""Causal calls whose workgroup size the kernel chooses from the lengths: what the rule says (CPU, the header's own functions compiled for the host) and
the results of either choice against the oracle (GPU)."""
import shutil
import subprocess

import numpy as np
import pytest

from paper_2508_11553_amd import build as sd_build
from tests.test_kernel_resources import CSRC

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "kernels.h"
struct Sequences {
    std::vector<int> nq, L;
    int tokens;
    int longest() const { int m = 0; for (size_t b = 0; b < L.size(); ++b) m = nq[b] > 0 && L[b] > m ? L[b] : m; return m; }
    int count(int t, int halves) const { return ((t << halves) + tokens - 1) / tokens; }
    template <class F> int total(F f) const { int n = 0; for (size_t b = 0; b < L.size(); ++b) n += nq[b] > 0 ? f(nq[b], L[b]) : 0; return n; }
};
int main(int argc, char **argv)
{
    const int units = atoi(argv[1]), heads = atoi(argv[2]), bound = atoi(argv[3]);
    Sequences s;
    s.tokens = 8 * units;
    int64_t total = 0;
    int most = 0, longest = 0;
    for (int i = 4; i + 1 < argc; i += 2) s.L.push_back(atoi(argv[i])), s.nq.push_back(atoi(argv[i + 1])), total += s.nq.back(), most = std::max(most, s.nq.back()), longest = std::max(longest, s.L.back());
    if (bound) most = bound;
    const int B = (int)s.L.size();
    const sd::PrefillPlan p = sd::prefill_plan(0, 128, total, most, B, heads, units, longest);
    printf("%d %d %d\n", p.blocks, sd::prefill_on_device(p, 0, 128, total, most, B, heads, units, longest), sd::prefill_prefers_four(s, heads, s.tokens));
}
"""

# (lens, queries, Hq, Hkv) and whether the kernel takes 4 blocks: edges of pages, tiles, pairs of pairs of tiles and workgroups' rows among the lengths, sequences
# without queries or tokens, more queries than tokens
EDGES = [0, 1, 15, 16, 17, 31, 33, 63, 65, 127, 129, 255, 257]
CASES = {
    "ragged": (([2600, 1700, 900, 300, 129, 33, 16, 1, 0, 700], [60, 50, 120, 100, 17, 33, 20, 1, 3, 0], 28, 4), True),
    "alike": (([1700, 1650, 1600, 1651, 1664, 1665, 1599, 1536], [100, 97, 96, 128, 100, 99, 100, 65], 32, 8), False),
    "many": ((EDGES * 4 + [1601, 1500, 777], [min(40, n) for n in EDGES * 4] + [90, 70, 50], 8, 2), True),
    "20 heads a group": (([1900, 1100, 1537, 64], [81, 60, 16, 50], 40, 2), True),
}


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    if shutil.which(sd_build.HIPCC) is None:
        pytest.skip("needs hipcc")
    d = tmp_path_factory.mktemp("on_device")
    (d / "choose.hip").write_text(PROGRAM)
    r = subprocess.run([sd_build.HIPCC, "--offload-host-only", "-std=c++17", f"-I{CSRC}", str(d / "choose.hip"), "-o", str(d / "choose")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def run(lens, nq, Hq, Hkv, bound=0):
        G = Hq // Hkv
        args = [16 // G if G <= 8 else 1, Hkv * ((G + 15) // 16), bound] + [x for pair in zip(lens, nq) for x in pair]
        got = subprocess.run([str(d / "choose")] + [str(x) for x in args], capture_output=True, text=True, check=True)
        return tuple(map(int, got.stdout.split()))
    return run


@pytest.mark.parametrize("name", CASES)
def test_the_cases_are_left_to_the_kernel(choose, name):
    call, four = CASES[name]
    blocks, on_device, prefers_four = choose(*call)
    assert blocks in (4, 8) and on_device and prefers_four == four


def test_ragged_calls_take_four_blocks_and_even_ones_eight(choose):
    assert choose([4092, 5323, 3358, 2488, 1434], [112, 20, 190, 274, 254], 28, 4)[1:] == (1, 1)   # 220 workgroups of 8 blocks, the longest sets the end
    assert choose([4000] * 4, [224] * 4, 28, 4)[1:] == (1, 0)                                       # 224 alike: one round
    assert choose([2000] * 4, [30] * 4, 64, 8)[2] == 1                                              # half a round of 8


def test_memory_bound_calls_are_not_read_twice(choose):
    """15 queries fit one workgroup of 8 blocks and need two of 4, both of which read the sequence's K/V."""
    assert choose([6800 + 383 * b for b in range(24)], [15] * 24, 64, 8)[1:] == (1, 0)
    assert choose([6800 + 383 * b for b in range(24)], [8] * 24, 64, 8)[1:] == (1, 1)     # one of 4
    assert choose([7601 + 32 * b for b in range(27)], [34] * 27, 16, 2)[1:] == (1, 0)     # 3 of 8, all at once
    assert choose([1963 + 60 * b for b in range(13)], [33] * 13, 32, 4)[1:] == (1, 0)


def test_calls_that_stay_with_the_host(choose):
    assert not choose([8000], [600], 28, 4)[1]                                  # one sequence: the bound is its length
    assert not choose([1500] * 5, [200] * 5, 28, 4)[1]                          # short contexts
    assert not choose([4000] * 65, [5] * 65, 28, 4)[1]                          # more sequences than lanes
    assert not choose([4092, 5323, 3358, 2488, 1434], [112, 20, 190, 274, 254], 28, 4, bound=1000)[1]   # a grid mostly empty


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_both_choices_against_the_oracle(name):
    import paper_2508_11553_amd as sd
    from tests.test_gpu_prefill import check, gpu, make, ref

    sd.load()
    (lens, nq, Hq, Hkv), _ = CASES[name]
    wl, q, q_start = make(lens, nq, Hq, Hkv, 128, seed=81)
    got = gpu(wl, q, q_start)
    assert not np.isnan(got).any()
    check(got, ref(wl, q, q_start))
