"""What the compiler made of the decode kernels (CPU only: hipcc cross-compiles for gfx950).

A kernel whose tile registers end up in scratch memory, or that no longer fits two waves per SIMD,
still computes the right thing and silently loses half its bandwidth, so the resource remarks of
the compiler are checked: the decode kernels (range pass, its probe, split pass, merge of the ranges) and the
causal kernels (the general one, the one in two phases, the one that loads straight into LDS; every instance of
them) use no scratch memory and spill no vector registers, and keep at least two waves per SIMD.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2508_11553_amd import build as sd_build

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2508_11553_amd", "csrc")


def resource_remarks(source, tmp_path):
    flags = [f for f in sd_build.FLAGS if f not in ("-shared", "-fPIC")]
    r = subprocess.run([sd_build.HIPCC, *flags, "--cuda-device-only", "-c", os.path.join(CSRC, source), "-o",
                        str(tmp_path / "dev.o"), "-Rpass-analysis=kernel-resource-usage"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    out, name = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"remark: .*Function Name: (\S+)", line)
        if m:
            name = m.group(1)
            out[name] = {}
            continue
        m = re.search(r"remark: \s*([A-Za-z ]+?)(?: \[[^\]]*\])?: (\d+)", line)
        if m and name:
            out[name][m.group(1).strip()] = int(m.group(2))
    return out


@pytest.mark.skipif(shutil.which(sd_build.HIPCC) is None and not os.path.exists(sd_build.HIPCC), reason="needs hipcc")
@pytest.mark.parametrize("source,kernels,least", [("attn_range.hip", "range_kernel", 8), ("attn_range.hip", "range_merge_kernel", 6),
                                                   ("attn_split.hip", "split_kernel", 10), ("attn_prefill.hip", "prefill_wide_kernel", 15),
                                                   ("attn_prefill.hip", "prefill_pingpong_kernel", 1), ("attn_prefill.hip", "prefill_direct_kernel", 3),
                                                   ("attn_prefill.hip", "prefill_wide_kernel_direct", 3), ("attn_prefill.hip", "prefill_wide_kernel_own", 3)])
def test_decode_kernels_keep_their_tiles_in_registers(source, kernels, least, tmp_path):
    remarks = {k: v for k, v in resource_remarks(source, tmp_path).items() if kernels in k}
    assert len(remarks) >= least, list(remarks)
    for name, res in remarks.items():
        assert res["ScratchSize"] == 0, (name, res)
        assert res["VGPRs Spill"] == 0, (name, res)
        # (three workgroups to a compute unit are what the small blocks of head_dim 64 gain by)
        assert res["Occupancy"] >= (3 if "prefill_direct_kernelILi64ELi4ELi2E" in name else 2), (name, res)


@pytest.mark.skipif(shutil.which(sd_build.HIPCC) is None and not os.path.exists(sd_build.HIPCC), reason="needs hipcc")
def test_a_compute_unit_holds_as_many_workgroups_of_the_split_pass_as_its_last_round_counts(tmp_path):
    """Workgroups of four waves, so waves per SIMD are workgroups per compute unit."""
    (tmp_path / "round.hip").write_text('#include <cstdio>\n#include "kernels.h"\nint main() { printf("%d %d", sd::split_round(64) / 256, sd::split_round(128) / 256); }\n')
    r = subprocess.run([sd_build.HIPCC, "--offload-host-only", "-std=c++17", f"-I{CSRC}", str(tmp_path / "round.hip"), "-o", str(tmp_path / "round")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    narrow, wide = map(int, subprocess.run([str(tmp_path / "round")], capture_output=True, text=True, check=True).stdout.split())
    remarks = {k: v for k, v in resource_remarks("attn_split.hip", tmp_path).items() if "split_kernel" in k}
    assert len(remarks) >= 10
    for name, res in remarks.items():
        assert res["Occupancy"] == (narrow if "Li64" in name or "Fp8Path64" in name else wide), (name, res)
