"""Causal calls of head_dim 128 over bf16 pools whose contexts stay under 512 tokens and whose workgroups of 16 column blocks are full, or not: which they are (CPU)
and both against the oracle (GPU).  Lengths lie on both sides of pages, tiles, rounds of two tiles and workgroups' rows; some sequences bring no queries, or more than
they have tokens."""
import numpy as np
import pytest

from tests.test_prefill_geometry import program, route  # noqa: F401  (program is a fixture)

LENS = [511, 300, 257, 256, 255, 129, 128, 127, 65, 64, 63, 33, 32, 31, 17, 16, 1, 0, 90]
CALLS = {   # (lens, queries, Hq, Hkv); whether the average sequence fills three quarters of a workgroup's blocks
    "whole prompts": ((LENS, LENS[:-1] + [120], 32, 8), True),
    "tails": ((LENS, [min(n, 70) if b != 4 else 0 for b, n in enumerate(LENS)], 42, 6), True),
    "20 heads a group": ((LENS[:9], [min(n, 40) for n in LENS[:9]], 80, 4), True),
    "few queries": ((LENS * 4, [min(n, 5) for n in LENS * 4], 8, 4), False),
}


@pytest.mark.parametrize("name", CALLS)
def test_the_calls_take_16_blocks_in_one_phase(program, name):  # noqa: F811
    (lens, nq, Hq, Hkv), full = CALLS[name]
    G = Hq // Hkv
    units = 16 // G if G <= 8 else 1
    got = route(program, lens, nq, Hq, Hkv, 128)
    assert got[:3] == (16, 1, 0) and got[4] == full
    assert (sum(nq) * 4 >= 16 * 3 * units * len(lens)) == full


@pytest.mark.gpu
@pytest.mark.parametrize("name", CALLS)
def test_both_kernels_against_the_oracle(name):
    import paper_2508_11553_amd as sd
    from tests.test_gpu_prefill import check, gpu, make, ref

    sd.load()
    (lens, nq, Hq, Hkv), _ = CALLS[name]
    wl, q, q_start = make(lens, nq, Hq, Hkv, 128, seed=93)
    check(gpu(wl, q, q_start), ref(wl, q, q_start))


@pytest.mark.gpu
@pytest.mark.parametrize("name", CALLS)
@pytest.mark.parametrize("what", ["negative scale", "zero scale", "constant V", "ramp", "jumps", "decay", "not finite past the end"])
def test_both_kernels_at_odd_scales_and_values(name, what):
    from tests.test_gpu_prefill import check, gpu, grow, make, poison, ref

    (lens, nq, Hq, Hkv), _ = CALLS[name]
    wl, q, q_start = make(lens, nq, Hq, Hkv, 128, seed=94, **{"negative scale": dict(scale=-0.11), "zero scale": dict(scale=0.0)}.get(what, {}))
    if what == "constant V":
        wl.v_pages[...] = 0x3ec0   # 0.375
        got, seen = gpu(wl, q, q_start), np.concatenate([np.arange(n) >= n - L for L, n in zip(lens, nq)])   # rows that see a token
        assert np.abs(got[seen] - 0.375).max() <= 2e-6 and not got[~seen].any()
        return
    if what in ("ramp", "jumps", "decay"):
        grow(wl, lens, what, "bf16")
    if what == "not finite past the end":
        poison(wl, lens)
    check(gpu(wl, q, q_start), ref(wl, q, q_start))
