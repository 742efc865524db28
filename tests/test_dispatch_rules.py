"""The host's rules that pick kernels and sizes (CPU only): the library's own functions, compiled for the host with
UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import pytest

from paper_2508_11553_amd import build as sd_build
from tests.test_kernel_resources import CSRC

PROGRAM = r"""
#include "api.hip"
#include <cstdio>
#include <cstdlib>
#include <cstring>
int main(int argc, char **argv)
{
    int v[16] = {};
    for (int i = 2; i < argc && i < 18; ++i) v[i - 2] = atoi(argv[i]);
    // batch, query heads, KV heads, head_dim, KV type, max_context_len come first
    const sd_shape s = {v[0], v[1], v[2], v[3], 16, 1, (v[5] + 15) / 16, v[4], v[5], 0};
    if (!strcmp(argv[1], "prefix_chunk")) {   // ... num_groups, max_group_size, max_shared_len
        const int c = prefix_chunk(&s, v[6], v[7], v[8]);
        printf("%d %d %d\n", c, pick_chunk(&s), ws_layout(&s, num_chunks(&s, c)).total <= sd_workspace_bytes(&s));
    } else if (!strcmp(argv[1], "short_enough")) {
        printf("%d\n", short_enough(&s));
    } else if (!strcmp(argv[1], "prefill_plan")) {   // ... total_q, max_q_len
        const int G = s.num_q_heads / s.num_kv_heads;
        const sd::PrefillPlan p = sd::prefill_plan(s.kv_dtype, s.head_dim, v[6], v[7], s.batch, s.num_kv_heads * sd::head_blocks(G), sd::units_per_block(G), s.max_context_len);
        printf("%d %d\n", p.blocks, p.split);
    } else if (!strcmp(argv[1], "stores")) {   // MB of rows, bytes beyond them, bytes of K/V per token and head
        const int64_t bytes = ((int64_t)v[6] << 20) + v[7];
        printf("%d %d %d\n", sd::stores_through(bytes), sd::window_tokens(bytes, s.max_context_len, v[8]), sd::split_round(s.head_dim) / 256);
    } else if (!strcmp(argv[1], "merge_width")) {   // items, rows, groups
        printf("%d\n", sd::merge_width(v[0], v[1], v[2]));
    }
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if shutil.which(sd_build.HIPCC) is None and not os.path.exists(sd_build.HIPCC):
        pytest.skip("needs hipcc")
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.hip").write_text(PROGRAM)
    # only host functions run, so the kernels' launch functions stay undefined
    r = subprocess.run([sd_build.HIPCC, "--offload-host-only", "-std=c++17", f"-I{CSRC}", "-Xarch_host", "-fsanitize=undefined",
                        "-Wl,--unresolved-symbols=ignore-all", str(d / "rules.hip"), "-o", str(d / "rules")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def call(*args):
        r = subprocess.run([str(d / "rules")] + [str(a) for a in args], capture_output=True, text=True, check=True)
        assert "runtime error" not in r.stderr, r.stderr
        return [int(x) for x in r.stdout.split()]
    return call


@pytest.mark.parametrize("shape,groups", [
    ((1500, 4, 1, 128, 0, 608), (2, 750, 448)),             # the slots of the chunk it would like do not fit the workspace
    ((64, 32, 8, 128, 0, 65536), (4, 2**31 - 1, 4096)),     # group bounds as loose as the type allows
    ((2**23, 8, 2, 128, 0, 2**21), (1, 16, 2**21)),         # chunks x sequences beyond 32 bits
    ((1, 1, 1, 64, 1, 16), (1, 1, 16)),
])
def test_prefix_chunk_stays_within_its_bounds(rule, shape, groups):
    chunk, from_shape, fits = rule("prefix_chunk", *shape, *groups)
    assert fits and 128 <= chunk <= from_shape


@pytest.mark.parametrize("shape,groups", [
    ((161, 40, 8, 64, 0, 411), (13, 20, 384)),       # a chunk or two per sequence
    ((46, 32, 4, 128, 0, 14880), (16, 5, 14048)),    # three quarters of the shape's chunk
])
def test_prefix_chunk_is_the_shape_s_where_a_shorter_one_does_not_pay(rule, shape, groups):
    chunk, from_shape, _ = rule("prefix_chunk", *shape, *groups)
    assert chunk == from_shape


def test_prefix_chunk_follows_the_groups(rule):
    chunk, from_shape, _ = rule("prefix_chunk", 56, 64, 8, 128, 0, 11500, 8, 7, 9000)
    assert 2 * chunk <= from_shape


@pytest.mark.parametrize("batch", [1, 16, 40, 64, 1024])
@pytest.mark.parametrize("kv_dtype,d,limit", [(0, 128, 1024), (0, 64, 1600), (1, 128, 1280), (1, 64, 1280)])
def test_single_pass_is_bounded_by_what_one_sequence_may_cost(rule, kv_dtype, d, limit, batch):
    """The lengths are not known here: one sequence of a batch may be as long as the bound and the rest empty, so the number of
    sequences must not move the line."""
    assert rule("short_enough", batch, 28, 4, d, kv_dtype, limit) == [1]
    assert rule("short_enough", batch, 28, 4, d, kv_dtype, limit + 1) == [0]


@pytest.mark.parametrize("items,rows,groups,width", [(512, 16, 1, 4), (2048, 16, 1, 4), (2048, 9, 1, 4), (2048, 8, 1, 2), (2048, 4, 1, 1),
                                                     (256, 16, 1, 1), (1024, 8, 1, 1), (2048, 16, 2, 1)])
def test_merge_pass_cuts_heads_only_where_items_are_few(rule, items, rows, groups, width):
    assert rule("merge_width", items, rows, groups) == [width]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("kv_dtype", [0, 1])
@pytest.mark.parametrize("batch,total_q,max_q", [(1, 1, 1), (1, 2**31 - 1, 2**31 - 1), (2**20, 2**31 - 1, 2**31 - 1), (2**20, 1, 1), (3, 100, 2**31 - 1)])
def test_prefill_plan_at_the_ends_of_its_arguments(rule, batch, total_q, max_q, kv_dtype, d):
    blocks, split = rule("prefill_plan", batch, 8, 2, d, kv_dtype, 2**21, total_q, max_q)
    assert (blocks, split) in {(16, 1), (8, 1), (8, 2), (4, 4), (2, 8)}
    if batch > 1:
        assert split <= 2   # a grid of more than 4096 workgroups takes the largest blocks there are


@pytest.mark.parametrize("d,kv,longest,mb,more,want", [
    (128, 0, 4096, 10, -16, [0, 0, 2]), (128, 0, 4096, 10, 0, [1, 256, 2]),      # 10 MB of rows
    (128, 0, 767, 32, 0, [1, 0, 2]), (128, 0, 768, 32, 0, [1, 256, 2]),          # 384 KB of K/V per head
    (128, 1, 1535, 32, 0, [1, 0, 2]), (128, 1, 1536, 32, 0, [1, 512, 2]),
    (64, 0, 1535, 32, 0, [1, 0, 4]), (64, 0, 1536, 32, 0, [1, 512, 4]),
    (64, 1, 3071, 32, 0, [1, 0, 4]), (64, 1, 3072, 32, 0, [1, 1024, 4]),
    (128, 0, 2**31 - 16, 2000, 0, [1, 256, 2]),                                  # bytes beyond 32 bits
])
def test_rows_that_are_written_through_and_in_windows(rule, d, kv, longest, mb, more, want):
    """Written through, tokens from which on a workgroup waits for a window, workgroups that a compute unit holds."""
    assert rule("stores", 1000, 64, 8, d, kv, longest, mb, more, 2 * d * (1 if kv else 2)) == want
