"""Which kernels a verify call runs, over its sizes and rules (CPU only)."""
import pytest

from paper_2405_19261_amd import spc
from paper_2405_19261_amd import workloads as W

SEQ, SMALL, TILES, TV_SELF, TV_PASS, TV_JOBS, JOBS, PAIR = (1 << i for i in range(8))
CUS = 256


def route(B, gamma, V, dtype, rules, per_seq=False, greedy=False):
    mask = sum(1 << r for r in rules)
    return spc.lib().spc_debug_route(B, gamma, V, spc.SPC_BF16 if dtype == "bf16" else
                                     spc.SPC_F32, mask, int(per_seq), int(greedy), CUS)


@pytest.mark.parametrize("args,want", [
    # the workloads
    ((1, 4, 1000, "f32", [W.CHOW]), SEQ),
    ((8, 5, 32128, "f32", [W.OPT]), TILES | TV_SELF),
    ((32, 7, 256000, "bf16", [W.DIFF]), TILES),
    ((128, 4, 256000, "bf16", [W.OPT], False, True), TILES | PAIR),
    ((256, 8, 256000, "bf16", [W.CHOW, W.DIFF, W.OPT], True), TILES | PAIR | TV_JOBS | JOBS),
    # second passes
    ((16, 7, 256000, "bf16", [W.OPT]), TILES | TV_PASS),
    ((32, 7, 256000, "bf16", [W.TOKEN_V2]), TILES | JOBS),
    ((8, 4, 20000, "bf16", [W.TOKEN_V2]), SMALL),
    # short sequences: one round of workgroups, and more
    ((8, 4, 2000, "bf16", [W.DIFF]), SEQ), ((8, 4, 2000, "bf16", [W.OPT]), SMALL),
    ((64, 7, 2000, "bf16", [W.OPT]), SEQ), ((64, 7, 3000, "bf16", [W.OPT]), SMALL),
    ((1024, 7, 1001, "bf16", [W.DIFF]), SEQ), ((1024, 7, 4097, "bf16", [W.DIFF]), TILES),
    ((600, 1, 2001, "f32", [W.TOKEN_V1]), SEQ), ((600, 1, 6401, "f32", [W.TOKEN_V1]), TILES | JOBS),
    ((8, 4, 1025, "bf16", [W.DIFF], False, True), SMALL),
    ((8, 4, 1024, "bf16", [W.DIFF], False, True), SEQ),
    # rows held by a workgroup: with first moments, and up to two rows a compute unit
    ((8, 4, 16384, "bf16", [W.DIFFLOG]), SMALL), ((8, 4, 16385, "bf16", [W.DIFFLOG]), TILES),
    ((8, 4, 24000, "bf16", [W.OPTLOG]), SMALL), ((8, 4, 24584, "bf16", [W.OPTLOG]), TILES | TV_SELF),
    ((8, 4, 8192, "bf16", [W.DIFF], False, True), SMALL),
    ((8, 4, 8193, "bf16", [W.DIFF], False, True), TILES),
    ((8, 4, 20480, "bf16", [W.DIFF]), SMALL), ((8, 4, 20481, "bf16", [W.DIFF]), TILES),
    ((50, 4, 20481, "bf16", [W.DIFF]), SMALL),
    ((100, 4, 12288, "bf16", [W.OPT]), SMALL), ((100, 4, 12289, "bf16", [W.OPT]), TILES | TV_PASS),
    # a resident grid with per-sequence rules takes its TV passes itself
    ((4, 4, 100000, "bf16", [W.DIFF, W.OPT], True), TILES | TV_SELF),
    # more tiles a row than its gate holds
    ((1, 1, 253952, "f32", [W.OPT]), TILES | TV_SELF),
    ((1, 1, 256000, "f32", [W.OPT]), TILES | TV_PASS),
    # sizes no call takes
    ((0, 4, 1000, "bf16", [W.DIFF]), 0), ((1, 64, 1000, "bf16", [W.DIFF]), 0),
    ((1, 4, 1, "bf16", [W.DIFF]), 0)])
def test_routes(args, want):
    assert route(*args) == want


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rule", range(13))
@pytest.mark.parametrize("greedy", [False, True])
def test_every_size_has_one_route(dtype, rule, greedy):
    """One way to the statistics and at most one to D_TV, at every size; a row
    of the one-launch paths fits them."""
    for B in (1, 2, 7, 64, 256, 300, 512, 513, 5000):
        for gamma in (1, 4, 15, 63):
            for V in (2, 7, 8, 1000, 4096, 16385, 32768, 32769, 256000, 2_000_001):
                r = route(B, gamma, V, dtype, [rule], greedy=greedy)
                assert bin(r & (SEQ | SMALL | TILES)).count("1") == 1
                tv = r & (TV_SELF | TV_PASS | TV_JOBS)
                assert bin(tv).count("1") <= 1
                if r & TILES and not greedy and rule in (W.OPT, W.OPTLOG):
                    assert tv
                if not r & TILES:
                    assert r in (SEQ, SMALL)
                    assert V <= (32768 if r == SEQ or dtype == "bf16" else 16384)
                    # (and no more rows than a launch's two a compute unit)
                    assert r == SEQ or B * (gamma + 1) <= 2 * CUS
