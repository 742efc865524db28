"""How the causal pass deals its items to the dies (CPU only): the header's own functions, compiled for the host."""
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
#include <cstring>
#include <vector>
#include "kernels.h"
int main(int argc, char **argv)
{
    if (!strcmp(argv[1], "split")) {
        const sd::SplitOrder o = sd::split_order(atoi(argv[2]), atoi(argv[3]), atoi(argv[4]));
        printf("%d %d\n", o.group, o.from);
        return 0;
    }
    if (argc > 3) {
        const int max_q = std::min(atoll(argv[8]), atoll(argv[2]));
        const sd::PrefillPlan p = sd::prefill_route(atoi(argv[7]), atoi(argv[1]), atoll(argv[2]), max_q, atoi(argv[3]), atoi(argv[4]), atoi(argv[5]), atoi(argv[6])).plan;
        const sd::PrefillPlan by_rule = sd::prefill_plan(atoi(argv[7]), atoi(argv[1]), atoll(argv[2]), max_q, atoi(argv[3]), atoi(argv[4]), atoi(argv[5]), atoi(argv[6]));
        printf("%d %d %d %d %d %d\n", p.on_device ? 0 : p.blocks, p.on_device ? 0 : p.split, p.phases, p.order, p.direct, by_rule.blocks);
        return 0;
    }
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


def block_case(blocks, d):
    """(lens, queries, Hq, Hkv): a small batch that the rule gives workgroups of `blocks` column blocks (bf16 pools), with sequences on both
    sides of a page, a tile, a round and a workgroup's rows."""
    edge = [1, 15, 16, 17, 31, 33, 129, 255, 256, 257]
    if d == 128:
        lens, q, Hq, Hkv = {16: (edge * 4 + [600], [1, 3, 17, 33] * 10 + [40], 16, 8),
                            8: ([700, 512, 400, 129, 33], [1000] * 5, 16, 8),
                            4: (edge[4:] + [700], [120] * 7, 16, 8),
                            2: (edge[4:] + [1030, 1500], [70] * 8, 8, 4)}[blocks]
    else:
        lens, q, Hq, Hkv = {16: ([129, 145, 160, 130] * 16 + edge, [160] * 74, 32, 32),
                            8: (edge + edge[2:], [1, 40, 130] * 6, 32, 32),
                            4: (edge[4:] + [700], [120] * 7, 16, 8),
                            2: (edge[4:] + [1030, 1500], [70] * 8, 8, 4)}[blocks]
    return lens, [min(n, L) for n, L in zip(q, lens)], Hq, Hkv


def context_bound(blocks, d):
    """The bound on the context lengths with which such a case of bf16 pools takes 16 blocks at head_dim 64; with their own lengths it takes 8."""
    return 1536 if (blocks, d) == (16, 64) else None


def stretch_case(plan, d):
    """(lens, queries, Hq, Hkv): sequences of 1500, 777 and 96 tokens, or many of 600, that take the plan (blocks, split, phases)."""
    long, many = [1500, 777, 96], [600] * 22 + [33, 511]
    return {
        (128, (16, 1, 1)): (long, [400, 400, 96], 64, 8),          # two phases
        (128, (16, 1, 0)): (many, [20] * 24, 32, 16),              # one phase: few queries per sequence
        (128, (8, 2, 0)): (long, [600, 777, 96], 16, 8),
        (128, (8, 1, 0)): ([511, 300, 96], [400, 300, 96], 16, 8),   # short contexts over fp8 pools
        (128, (4, 4, 0)): (long, [400, 200, 96], 16, 8),
        (128, (2, 8, 0)): (long, [100, 77, 96], 8, 2),
        (64, (16, 1, 0)): ([700, 450, 320, 129] * 16, [128] * 64, 64, 32),
        (64, (8, 1, 0)): (long * 3, [400, 400, 96] * 3, 16, 8),
        (64, (4, 4, 0)): (long, [400, 777, 96], 16, 8),
        (64, (2, 8, 0)): (long, [100, 77, 96], 8, 2),
    }[d, plan]


PLANS = [("bf16", 128, (16, 1, 1))] + [(kv, 128, p) for kv in ("bf16", "fp8") for p in ((16, 1, 0), (8, 2, 0), (4, 4, 0), (2, 8, 0))] + \
    [("fp8", 128, (8, 1, 0)), ("bf16", 64, (16, 1, 0))] + [(kv, 64, p) for kv in ("bf16", "fp8") for p in ((8, 1, 0), (4, 4, 0), (2, 8, 0))]


def plan(program, lens, q, Hq, Hkv, d, kv_dtype="bf16", bound=None, max_q=None):
    """(column blocks of a workgroup, waves that share a block's range, two phases) of a call as it runs; (0, 0, 0) where the kernel chooses 8 or 4."""
    return route(program, lens, q, Hq, Hkv, d, kv_dtype, bound, max_q)[:3]


def plan_and_order(program, lens, q, Hq, Hkv, d, kv_dtype="bf16", bound=None, max_q=None):
    """The same and the classes of the order in which the workgroups start, 0: dealt pair by pair."""
    return route(program, lens, q, Hq, Hkv, d, kv_dtype, bound, max_q)[:4]


def route(program, lens, q, Hq, Hkv, d, kv_dtype="bf16", bound=None, max_q=None):
    """The same, whether 16 blocks load straight into LDS in one phase, and the blocks that the host's rule gives where the kernel does not choose."""
    G = Hq // Hkv
    args = (d, sum(q), len(lens), Hkv * ((G + 15) // 16), 16 // G if G <= 8 else 1, bound or max(lens), int(kv_dtype == "fp8"), max_q or max(q))
    got = subprocess.run([program] + [str(x) for x in args], capture_output=True, text=True, check=True)
    return tuple(int(x) for x in got.stdout.split())


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("blocks", [16, 8, 4, 2])
def test_the_block_cases_are_what_they_say(program, blocks, d):
    assert plan(program, *block_case(blocks, d), d, bound=context_bound(blocks, d))[0] == blocks


@pytest.mark.parametrize("kv_dtype,d,want", PLANS)
def test_the_stretch_cases_are_what_they_say(program, kv_dtype, d, want):
    assert plan(program, *stretch_case(want, d), d, kv_dtype, context_bound(want[0], d)) == want


@pytest.mark.parametrize("call", [block_case(16, 64), stretch_case((16, 1, 0), 64)])
def test_the_cases_of_16_blocks_at_head_dim_64_take_8_with_their_own_lengths(program, call):
    assert plan(program, *call, 64) == (8, 1, 0)


def test_two_phases_only_where_most_waves_have_rows(program):
    """49 sequences with a query or two each: the waves without rows would take their turn at the matrix pipe all the same."""
    assert plan(program, [43] * 24 + [2539] * 25, [1] * 49, 128, 4, 128)[2] == 0
    assert plan(program, [8192] * 16, [2048] * 16, 32, 8, 128) == (16, 1, 1)


def test_workgroups_that_fill_the_chip_are_not_cut_further(program):
    assert plan(program, [60] * 59 + [1185], [49] * 60, 8, 2, 64, bound=18960)[0] == 4
    assert plan(program, [348] * 18, [32] * 18, 32, 4, 64, bound=1392)[0] >= 4


def test_16_blocks_at_head_dim_64_are_for_bf16_pools_and_full_workgroups(program):
    assert plan(program, [1500] * 50, [280] * 50, 128, 4, 64, "fp8") == (8, 1, 0)
    assert plan(program, [92] * 61, [15] * 61, 32, 32, 64) == (8, 1, 0)
    assert plan(program, [3000] * 8, [3000] * 8, 32, 8, 64) == (16, 1, 0)


def test_a_loose_bound_on_the_queries_keeps_the_grid_small(program):
    lens, q = [76] * 55, [23] * 54 + [45]
    assert plan(program, lens, q, 4, 1, 128, bound=548) == (4, 4, 0)
    assert plan(program, lens, q, 4, 1, 128, bound=548, max_q=sum(q)) == (8, 2, 0)
    assert plan(program, [76] * 110, [12] * 110, 4, 1, 128, bound=548) == (4, 4, 0)
    assert plan(program, [76] * 110, [12] * 110, 4, 1, 128, bound=548, max_q=12 * 110)[0] == 16
    assert plan(program, [2000] * 64, [40] * 64, 8, 2, 64)[0] == 4
    assert plan(program, [2000] * 64, [40] * 64, 8, 2, 64, max_q=40 * 64)[0] == 8


EDGES = [1, 16, 31, 32, 33, 63, 65, 127, 128, 129, 255, 257, 290]   # contexts that end at pages, tiles and rounds of 2, 4 and 8 tiles


def direct_case(blocks, short, d):
    """(lens, queries, Hq, Hkv) over bf16 pools that take 8, 4 or 2 column blocks, with contexts below 512 tokens or not."""
    Hq, Hkv, most = {8: (28, 4, 75), 4: (28, 4, 30), 2: (8, 2, 20)}[blocks]
    lens = EDGES + [300 if short else 777]
    return lens, [min(L, most) for L in lens], Hq, Hkv


DIRECT = [(128, blocks, short) for blocks in (8, 4, 2) for short in (True, False)] + [(64, 4, False), (64, 2, True), (64, 2, False)]


@pytest.mark.parametrize("d,blocks,short", DIRECT)
def test_short_and_longer_contexts_take_every_split(program, d, blocks, short):
    assert plan(program, *direct_case(blocks, short, d), d) == (blocks, 16 // blocks, 0)


@pytest.mark.parametrize("batch,blocks", [(11, 8), (12, 16), (15, 16), (16, 16), (17, 8), (19, 8), (20, 16)])
def test_one_round_of_large_workgroups_stays_and_a_few_more_are_cut(program, batch, blocks):
    """Long contexts over bf16 pools: 16 workgroups per sequence, 256 of which run at once."""
    assert route(program, [4000] * batch, [96] * batch, 32, 8, 128)[5] == blocks


@pytest.mark.parametrize("batch,blocks", [(22, 16), (32, 16), (33, 8), (34, 8), (39, 8), (40, 16)])
def test_one_round_is_counted_by_full_blocks_where_all_are_full(program, batch, blocks):
    """8 workgroups per sequence without an empty row."""
    assert route(program, [4000] * batch, [64] * batch, 32, 8, 128)[5] == blocks


@pytest.mark.parametrize("q,blocks", [(176, 4), (184, 8), (216, 8), (232, 8)])
def test_long_contexts_over_bf16_pools_are_cut_below_8_blocks_where_192_workgroups_are_not_reached(program, q, blocks):
    """Two sequences of long contexts: 184, 192, 224 and 240 workgroups of 8 blocks.  (The host's rule; with bounds as tight as these the kernel chooses.)"""
    assert route(program, [8000] * 2, [q] * 2, 64, 8, 128)[5] == blocks
    assert plan(program, [8000] * 2, [q] * 2, 64, 8, 128) == (0, 0, 0)


LONGEST_FIRST = [(6, 2, 128, "bf16"), (4, 4, 64, "bf16"), (8, 2, 128, "fp8")]


def longest_first_case(B, Hq, Hkv, d):
    """(lens, queries, Hq, Hkv) of batches with two long sequences; larger ones also have sequences without queries, with more queries than tokens, and
    empty ones."""
    if B == 2:
        return [2300 if d == 64 else 1500, 1100], [1400, 1100], *((16, 16) if d == 64 else (Hq, Hkv))
    rng = np.random.default_rng(B)
    lens = [1100, 530] + [int(x) for x in rng.integers(0, 300, B - 2)]
    nq = [700, 530] + [int(x) for x in rng.integers(0, 60, B - 2)]
    lens[5], nq[5], nq[6], nq[7] = 0, 9, 0, lens[7] + 20
    return lens, nq, Hq, Hkv


@pytest.mark.parametrize("B,classes", [(2, 8), (64, 8), (65, 0)])
@pytest.mark.parametrize("Hq,Hkv,d,kv_dtype", LONGEST_FIRST)
def test_the_longest_first_cases_are_what_they_say(program, Hq, Hkv, d, kv_dtype, B, classes):
    blocks, _, _, order = plan_and_order(program, *longest_first_case(B, Hq, Hkv, d), d, kv_dtype)
    assert order == classes and blocks   # not left to the kernel


FOUR_CLASSES = ([1300, 1200, 1250, 700, 330, 1300, 1100, 40], [1300, 900, 1250, 700, 200, 1100, 1100, 40], 32, 32, 64)   # ragged


@pytest.mark.parametrize("call,want", [(FOUR_CLASSES, (8, 1, 0, 4)), (([8000] * 8, [2048] * 8, 32, 8, 128), (16, 1, 1, 4)),
                                       (([8000] * 8, [1100] * 8, 32, 8, 128), (16, 1, 1, 8))])
def test_large_calls_are_ordered_in_four_classes(program, call, want):
    assert plan_and_order(program, *call) == want


@pytest.mark.parametrize("lens,q,classes", [([8000], [4096], 0), ([1500, 1400], [512, 512], 0), ([1500, 1400], [528, 512], 8)])
def test_single_sequences_and_calls_that_run_at_once_are_dealt(program, lens, q, classes):
    """Workgroups of 32 queries, 256 of which run at once."""
    assert plan_and_order(program, lens, q, 32, 8, 128) == ((16, 1, 1) if len(lens) == 1 else (8, 2, 0)) + (classes,)


@pytest.mark.parametrize("lens,q,Hq,Hkv,d,classes", [
    ([799] * 8, [780] * 8, 40, 8, 128, 0),            # 4 rounds of 256 workgroups, contexts worth 3
    ([799] * 5, [780] * 5, 40, 8, 128, 8),            # 2.6
    ([799] * 5, [780] * 5, 40, 8, 64, 0),             # head_dim 64, contexts under 1024: 1.7 rounds of 768, one at most
    ([799] * 20, [20] * 19 + [400], 12, 12, 64, 8),   # 0.5; the bound on the queries leaves room for more
    ([1024] * 5, [780] * 5, 40, 8, 64, 8),
    ([8192] * 15, [2048] * 15, 32, 8, 128, 4),        # 15.2 rounds
    ([8192] * 16, [2048] * 16, 32, 8, 128, 0),        # 16.3
])
def test_longest_first_only_where_the_rounds_are_few_for_the_context(program, lens, q, Hq, Hkv, d, classes):
    assert plan_and_order(program, lens, q, Hq, Hkv, d)[3] == classes


@pytest.mark.parametrize("batch,q,heads,d,kv_dtype,classes", [
    (24, 58, (8, 2), 128, "bf16", 0), (24, 58, (8, 2), 64, "bf16", 0), (24, 58, (8, 2), 128, "fp8", 8), (24, 29, (28, 4), 64, "bf16", 0),
    (24, 29, (32, 8), 64, "bf16", 8), (12, 80, (8, 2), 128, "bf16", 0), (11, 90, (8, 2), 128, "bf16", 8), (11, 60, (28, 4), 64, "bf16", 8)])
def test_two_block_workgroups_over_bf16_pools_of_many_sequences_are_ordered_only_where_a_head_keeps_its_die(program, batch, q, heads, d, kv_dtype, classes):
    assert plan_and_order(program, [6000 + 20 * b for b in range(batch)], [q * (3 + b % 2 * 5) // 8 for b in range(batch)], *heads, d, kv_dtype) == (2, 8, 0, classes)


LONGEST_FIRST_ITEMS = {   # (sequences, longest): sequences of a group, the first that belongs to one; 4 KV heads
    (513, 1100): (256, 257),   # the batch's last sequences only
    (600, 2100): (256, 0),     # all of them, 88 + 256 + 256
    (256, 2100): (256, 0),     # a single group
}


@pytest.mark.parametrize("batch,heads,longest,want", [(b, 4, n, w) for (b, n), w in LONGEST_FIRST_ITEMS.items()] + [
    (300, 2, 1024, (256, 44)), (300, 2, 2048, (256, 0)),   # behind shared prefixes, chunks of 1024 and 2048
    (128, 4, 4096, (256, 128)), (129, 4, 4096, (256, 0)),  # all workgroups run at once, and one sequence more
    (600, 4, 1023, (256, 600)), (600, 64, 1024, (64, 536)), (600, 4096, 2048, (64, 0)), (200, 4, 1024, (256, 0)),
])
def test_order_of_the_split_pass(program, batch, heads, longest, want):
    got = subprocess.run([program, "split", str(batch), str(heads), str(longest)], capture_output=True, text=True, check=True)
    assert tuple(map(int, got.stdout.split())) == want
