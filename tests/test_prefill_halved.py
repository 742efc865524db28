"""Causal calls of head_dim 64 over bf16 pools whose plan is 16 column blocks: 8 where no sequence may reach 1536 tokens.  The rule (CPU, the header's own
functions compiled for the host) and both sizes on the same batches against the oracle (GPU)."""
import shutil
import subprocess

import pytest

from paper_2508_11553_amd import build as sd_build
from tests.test_kernel_resources import CSRC
from tests.test_prefill_geometry import block_case, stretch_case

PROGRAM = r"""
#include <cstdio>
#include "kernels.h"
int main()
{
    for (int kv : {0, 1})
        for (int d : {64, 128})
            for (int blocks : {16, 8, 4, 2})
                for (int longest : {100, 1535, 1536, 100000}) printf("%d %d %d %d %d\n", kv, d, blocks, longest, sd::prefill_halved(sd::PrefillPlan{blocks, 1, false}, kv, d, 8000, 1000, 16, 8, 4, longest).blocks);
    for (int bound : {500, 1000, 1100, 5000}) printf("%d\n", sd::prefill_halved(sd::PrefillPlan{16, 1, false}, 0, 64, 8000, bound, 16, 8, 4, 1000).blocks);
}
"""


@pytest.mark.skipif(shutil.which(sd_build.HIPCC) is None, reason="needs hipcc")
def test_only_plans_of_16_at_head_dim_64_over_bf16_pools_are_halved(tmp_path):
    (tmp_path / "halved.hip").write_text(PROGRAM)
    r = subprocess.run([sd_build.HIPCC, "--offload-host-only", "-std=c++17", f"-I{CSRC}", str(tmp_path / "halved.hip"), "-o", str(tmp_path / "halved")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = subprocess.run([str(tmp_path / "halved")], capture_output=True, text=True, check=True).stdout.splitlines()
    assert len(lines) == 68
    assert lines[64:] == ["8", "8", "16", "16"]   # queries of a sequence, bound; the average is 500: no grid that is mostly empty
    for line in lines[:64]:
        kv, d, blocks, longest, got = map(int, line.split())
        assert got == (8 if (kv, d, blocks) == (0, 64, 16) and longest < 1536 else blocks)


@pytest.mark.gpu
@pytest.mark.parametrize("bound", [None, 1535, 1536])
@pytest.mark.parametrize("case", ["stretch", "edges"])
def test_both_sizes_against_the_oracle(case, bound):
    import paper_2508_11553_amd as sd
    from tests.test_gpu_prefill import check_first, make

    sd.load()
    lens, nq, Hq, Hkv = stretch_case((16, 1, 0), 64) if case == "stretch" else block_case(16, 64)
    wl, q, q_start = make(lens, nq, Hq, Hkv, 64, seed=87, max_blocks_per_seq=256)
    if bound:
        wl.max_context_len = bound
    check_first(wl, q, q_start, 4 if case == "stretch" else 8, "bf16")
