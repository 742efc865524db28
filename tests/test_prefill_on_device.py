"""Causal calls whose workgroup size the kernel chooses from the lengths: what the rule says (CPU, the header's own functions compiled for the host) and
the results of either choice against the oracle (GPU)."""
import shutil
import subprocess

import numpy as np
import pytest

from paper_2508_11553_amd import build as sd_build
from tests.test_kernel_resources import CSRC
from tests.test_prefill_geometry import plan, program  # noqa: F401  (program is a fixture)

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


# 120 workgroups of 8 blocks and 200 of 4; 240 and 400
LEVEL = {5: True, 10: False}


@pytest.mark.parametrize("B", LEVEL)
def test_what_the_kernel_takes_for_level_calls(choose, B):
    assert choose([1600] * B, [150] * B, 16, 8)[1:] == (1, LEVEL[B])


# (lens, queries), whether the kernel takes 4 blocks.  The first sequence alone is the host's: 8 blocks under its own bound on the length, 4 under 2048
ALONE = {"ragged": ([1990, 200], [590, 200], True), "alike": ([1990, 1980], [640, 640], False)}


@pytest.mark.parametrize("name", ALONE)
def test_the_first_sequence_alone_takes_either_size(choose, program, name):  # noqa: F811
    lens, nq, four = ALONE[name]
    assert choose(lens, nq, 28, 4)[2] == four
    assert plan(program, lens, nq, 28, 4, 128, bound=4096) == (0, 0, 0)
    assert plan(program, lens[:1], nq[:1], 28, 4, 128) == (8, 2, 0) and plan(program, lens[:1], nq[:1], 28, 4, 128, bound=2048) == (4, 4, 0)


@pytest.mark.gpu
@pytest.mark.parametrize("name", ALONE)
def test_the_size_that_runs_is_the_one_the_lengths_ask_for(name):
    """Bit for bit the rows of the first sequence by the host's kernel of that size, and not those of the other."""
    from tests.test_gpu_prefill import gpu, make_bound

    lens, nq, four = ALONE[name]
    wl, q, q_start = make_bound(lens, nq, 28, 4, 128, "bf16", 4096, seed=82)
    rows = q_start[1]
    got = gpu(wl, q, q_start)[:rows]
    wl.batch, wl.block_table, wl.context_lens = 1, wl.block_table[:1], wl.context_lens[:1]
    by_size = {}
    for size, bound in ((8, lens[0]), (4, 2048)):
        wl.max_context_len = bound
        by_size[size] = gpu(wl, q[:rows], q_start[:2])
    assert np.array_equal(got, by_size[4 if four else 8])
    assert not np.array_equal(by_size[4], by_size[8])


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("what", ["plain", "negative scale", "zero scale", "constant V", "ramp", "jumps", "decay", "not finite past the end"])
def test_both_choices_against_the_oracle(name, what):
    import paper_2508_11553_amd as sd
    from tests.test_gpu_prefill import check, gpu, grow, make, poison, ref

    sd.load()
    (lens, nq, Hq, Hkv), _ = CASES[name]
    wl, q, q_start = make(lens, nq, Hq, Hkv, 128, seed=81, **{"negative scale": dict(scale=-0.11), "zero scale": dict(scale=0.0)}.get(what, {}))
    if what == "constant V":
        wl.v_pages[...] = 0x3ec0   # 0.375
        got, seen = gpu(wl, q, q_start), np.concatenate([np.arange(n) >= n - L for L, n in zip(lens, nq)])   # rows that see a token
        assert np.abs(got[seen] - 0.375).max() <= 2e-6 and not got[~seen].any()
        return
    if what in ("ramp", "jumps", "decay"):
        grow(wl, lens, what, "bf16")
    if what == "not finite past the end":
        poison(wl, lens)
    got = gpu(wl, q, q_start)
    assert not np.isnan(got).any()   # every row was written
    check(got, ref(wl, q, q_start))


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_looser_bounds_change_nothing(name, choose):
    from tests.test_gpu_prefill import gpu, make_bound

    (lens, nq, Hq, Hkv), _ = CASES[name]
    wide = max(nq) + 4   # more slots of a sequence in all but one
    assert choose(lens, nq, Hq, Hkv, bound=wide)[1:] == choose(lens, nq, Hq, Hkv)[1:]
    wl, q, q_start = make_bound(lens, nq, Hq, Hkv, 128, "bf16", 6000, seed=83)
    loose = gpu(wl, q, q_start, max_q=wide)
    wl.max_context_len = max(lens)
    assert np.array_equal(loose, gpu(wl, q, q_start))


@pytest.mark.gpu
@pytest.mark.parametrize("name", CASES)
def test_ranges_outside_of_the_rows_are_skipped(name):
    from tests.test_gpu_prefill import check, gpu, make, ref

    (lens, nq, Hq, Hkv), _ = CASES[name]
    wl, q, q_start = make(lens, nq, Hq, Hkv, 128, seed=84)
    last = max(b for b, n in enumerate(nq) if n)   # its range is to end behind the rows, that of the first sequence to begin before them
    bad = q_start.copy()
    bad[0], bad[last + 1:] = -3, len(q) + 8
    got = gpu(wl, q, bad, max_q=max(nq) + 8)
    inner = slice(q_start[1], q_start[last])
    assert np.isnan(got[:q_start[1]]).all() and np.isnan(got[q_start[last]:]).all()
    check(got[inner], ref(wl, q, q_start)[inner])


@pytest.mark.gpu
@pytest.mark.parametrize("B", LEVEL)
def test_later_tokens_that_are_not_finite_do_not_reach_earlier_rows(B):
    """K and V rows of the last 20 tokens: rows that end a tile and a wave's rows before them do not change."""
    from tests.test_gpu_prefill import gpu, make

    L, n = 1600, 150
    wl, q, q_start = make([L] * B, [n] * B, 16, 8, 128, seed=85)
    want = gpu(wl, q, q_start)
    for b in range(B):
        for t in range(L - 20, L):
            wl.v_pages[wl.block_table[b, t // 16], :, t % 16] = 0x7fc0 if t % 2 else 0x7f80
            wl.k_pages[wl.block_table[b, t // 16], :, t % 16] = 0x7fc0 if t % 3 else 0xff80
    got = gpu(wl, q, q_start)
    assert np.array_equal(got.reshape(B, n, -1)[:, :n - 84], want.reshape(B, n, -1)[:, :n - 84])
