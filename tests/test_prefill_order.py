"""In which order the causal pass starts the query blocks of a batch (CPU only): the header's own functions, compiled for the host with
the sequences walked one by one where the kernel has one in every lane."""
import random
import shutil
import subprocess

import pytest

from paper_2508_11553_amd import build as sd_build
from tests.test_kernel_resources import CSRC

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>
#include "kernels.h"
struct Sequences {
    std::vector<int> end, blocks;
    struct Found { int b, before, end, blocks; };
    int top() const { int m = 0; for (int e : end) m = e > m ? e : m; return m; }
    template <class F> int sum(F f) const { int n = 0; for (size_t b = 0; b < end.size(); ++b) n += f(end[b], blocks[b]); return n; }
    template <class F> Found find(F f, int m) const
    {
        int before = 0;
        for (size_t b = 0; b < end.size(); ++b) {
            const int n = f(end[b], blocks[b]);
            if (before + n > m) return Found{(int)b, before, end[b], blocks[b]};
            before += n;
        }
        exit(3);
    }
};
int main(int argc, char **argv)
{
    if (argc == 2) {   // the reciprocal of every size of a workgroup, where it could first go wrong
        long bad = 0;
        for (unsigned t = 1; t <= 256; ++t) {
            const uint32_t r = sd::reciprocal_of(t);
            for (unsigned q = 1; t > 1 && q < (1u << 24) / t; q += q < 64 ? 1 : q / 7) bad += (uint64_t)(q * t) * r >> 32 != q || (uint64_t)(q * t - 1) * r >> 32 != q - 1;
        }
        printf("%ld\n", bad);
        return 0;
    }
    if (!strcmp(argv[1], "slots")) {   // heads, slots of a (sequence, head) pair; what every workgroup of the grid takes
        Sequences s;
        for (int i = 4; i + 1 < argc; i += 2) s.end.push_back(atoi(argv[i])), s.blocks.push_back(atoi(argv[i + 1]));
        const int heads = atoi(argv[2]), slots = (int)s.end.size() * heads * atoi(argv[3]);
        for (int i = 0; i < (slots + 7) / 8 * 8; ++i) {
            const sd::PrefillSlot p = sd::prefill_slot(s, i, heads);
            if (p.block >= 0) printf("%d %d %d %d\n", i, p.b, p.head, p.block);
        }
        return 0;
    }
    const int classes = atoi(argv[1]);
    Sequences s;
    for (int i = 2; i + 1 < argc; i += 2) s.end.push_back(atoi(argv[i])), s.blocks.push_back(atoi(argv[i + 1]));
    for (int k = 0;; ++k) {
        const sd::PrefillBlock p = sd::prefill_pick(s, k, classes);
        if (p.block < 0) break;
        printf("%d %d\n", p.b, p.block);
    }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which(sd_build.HIPCC) is None:
        pytest.skip("needs hipcc")
    d = tmp_path_factory.mktemp("order")
    (d / "order.hip").write_text(PROGRAM)
    r = subprocess.run([sd_build.HIPCC, "--offload-host-only", "-std=c++17", f"-I{CSRC}", "-Xarch_host", "-fsanitize=undefined", str(d / "order.hip"), "-o", str(d / "order")],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return str(d / "order")


def sequences(kind, rng):
    """[(where the last block ends, blocks)]: a sequence may have no queries, or more of them than tokens."""
    return {"one": [(7, 3)],
            "equal": [(32, 8)] * 16,
            "edges": [(0, 0), (5, 5), (1, 4), (0, 2), (64, 1), (63, 63), (8, 0), (40, 41)],
            "64": [(rng.randint(0, 200), rng.randint(0, 60)) for _ in range(64)],
            "long": [(1 << 20, 3), ((1 << 20) - 9, 200), (1, 1)]}[kind]


@pytest.mark.parametrize("classes", [4, 8])
@pytest.mark.parametrize("kind", ["one", "equal", "edges", "64", "long"])
def test_every_block_once_and_longest_first(program, kind, classes):
    seqs = sequences(kind, random.Random(3))
    args = [str(x) for e in seqs for x in e]
    got = [tuple(map(int, l.split())) for l in subprocess.run([program, str(classes)] + args, capture_output=True, text=True, check=True).stdout.splitlines()]
    assert sorted(got) == sorted((b, j) for b, (_, n) in enumerate(seqs) for j in range(n))
    top = max(e for e, _ in seqs)
    edges = [top * c // classes for c in range(1, classes)]
    of = [sum(seqs[b][0] - (seqs[b][1] - 1 - j) > e for e in edges) for b, j in got]   # the class of a block's end
    assert of == sorted(of, reverse=True)
    for a, b in zip(zip(of, got), list(zip(of, got))[1:]):   # within a class: sequence after sequence, late blocks first
        if a[0] == b[0]:
            assert a[1][0] < b[1][0] or (a[1][0] == b[1][0] and a[1][1] == b[1][1] + 1)


def test_the_reciprocal_divides_exactly(program):
    assert subprocess.run([program, "-"], capture_output=True, text=True, check=True).stdout == "0\n"


@pytest.mark.parametrize("heads", [1, 2, 4, 8, 12, 16])
@pytest.mark.parametrize("kind", ["one", "edges", "few", "64", "equal"])
def test_workgroups_of_calls_whose_size_the_kernel_chooses(program, kind, heads):
    """Every block of every head once; where all run at once and a head would not keep its die, as many on every die and a pair on one die, but for 7."""
    seqs = {"few": [(90, 3), (12, 1), (70, 5), (33, 2), (8, 2)]}.get(kind) or sequences(kind, random.Random(7))
    args = [str(x) for e in seqs for x in e]
    lines = subprocess.run([program, "slots", str(heads), str(max(n for _, n in seqs))] + args, capture_output=True, text=True, check=True).stdout.splitlines()
    got = [tuple(map(int, l.split())) for l in lines]
    n = sum(b for _, b in seqs) * heads
    assert sorted(g[1:] for g in got) == sorted((b, h, j) for b, (_, blocks) in enumerate(seqs) for h in range(heads) for j in range(blocks))
    if heads % 8 == 0 or n > 256:
        order = [tuple(map(int, l.split())) for l in subprocess.run([program, "8"] + args, capture_output=True, text=True, check=True).stdout.splitlines()]
        assert [g[1:] for g in got] == [(b, h, j) for b, j in order for h in range(heads)]
        return
    dies = [[g[1:3] for g in got if g[0] % 8 == die] for die in range(8)]
    assert max(map(len, dies)) <= -(-n // 8)
    assert sum(len(set(d)) for d in dies) <= len({g[1:3] for g in got}) + 7
