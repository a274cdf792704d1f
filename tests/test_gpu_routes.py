"""The kernels' routes at the sizes where each can go wrong, against the fp64
oracle (needs an MI355X)."""
import numpy as np
import pytest
import torch

import oracle
import parity
from paper_2405_19261_amd import spc
from paper_2405_19261_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()


# Bits of spc_debug_route.
SEQ, SMALL, TILES, TV_SELF, TV_PASS, TV_JOBS, JOBS, PAIR = (1 << i for i in range(8))


def route(B, gamma, V, dtype, rule, greedy=False, per_seq=False):
    """The kernels a call of these sizes runs on this device."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return spc.lib().spc_debug_route(B, gamma, V, spc.SPC_BF16 if dtype == "bf16" else
                                     spc.SPC_F32, 1 << rule, int(per_seq), int(greedy), cus)


def check(inp, dtype, greedy=False, stats=True, per_seq=False):
    """One call against the oracle; returns the GPU's outputs."""
    g = parity.run_gpu(inp, greedy=greedy, stats=stats, per_seq=per_seq)
    h = parity.host_inputs(inp)
    parity.compare(g, parity.run_oracle(h, greedy=greedy), h, dtype, greedy=greedy)
    return g


# Rows that start inside a 16-byte vector and end inside a lane load: fewer
# entries than one vector, one entry either side of a vector, of a
# wavefront's lane load and of a tile (8192 bfloat16 / 4096 float32), on the
# statistics-tile path (more sequences than the one-launch paths take, or
# rows longer than theirs) with each of its second passes; sampled rows that
# another path takes are greedy here.
@pytest.mark.parametrize("dtype,V,B,rule,want", [
    ("bf16", 2, 600, W.DIFF, None), ("bf16", 7, 600, W.OPT, None),
    ("bf16", 9, 600, W.TOKEN_V2, None), ("bf16", 511, 600, W.LOSSY, None),
    ("bf16", 513, 600, W.OPT, None), ("bf16", 2049, 600, W.OPT, TV_PASS),
    ("bf16", 2049, 600, W.DIFFLOG, 0), ("bf16", 3601, 600, W.OPTLOG, TV_PASS),
    ("bf16", 8191, 560, W.DIFF, 0), ("bf16", 8193, 560, W.TOKEN_V1, JOBS),
    ("bf16", 40001, 5, W.OPT, TV_SELF), ("bf16", 40001, 5, W.TOKEN_V2, JOBS),
    ("bf16", 65543, 70, W.DIFF, 0), ("bf16", 65543, 40, W.OPT, TV_PASS),
    ("f32", 3, 600, W.DIFF, 0), ("f32", 5, 600, W.OPT, TV_PASS), ("f32", 5, 600, W.OPTLOG, TV_PASS),
    ("f32", 255, 600, W.DIFFLOG, 0), ("f32", 257, 600, W.OPT, TV_PASS),
    ("f32", 6401, 600, W.TOKEN_V3, JOBS),
    ("f32", 4095, 560, W.BILD, 0), ("f32", 4097, 560, W.DIFFLOG, 0),
    ("f32", 33333, 6, W.OPTLOG, TV_SELF), ("f32", 33333, 40, W.OPTLOG, TV_PASS)])
@pytest.mark.parametrize("greedy", [False, True])
def test_rows_at_any_alignment(dtype, V, B, rule, want, greedy):
    passes = TV_SELF | TV_PASS | TV_JOBS | JOBS
    greedy = greedy or want is None
    r = route(B, 1, V, dtype, rule, greedy)
    assert r & TILES and (greedy or r & passes == want), r
    wl = W.WORKLOADS[3].with_(B=B, gamma=1, V=V, dtype=dtype, rule=rule, alpha=0.1,
                              temperature=0.0 if greedy else 1.0)
    parity.parity_workload(wl, 1, step0=31, report_name=f"anyalign.{dtype}.{V}")


@pytest.mark.parametrize("dtype,V,B,rule", [("bf16", 8193, 560, W.OPT), ("bf16", 40001, 70, W.OPT),
                                            ("f32", 33333, 70, W.OPTLOG)])
def test_tv_jobs_at_any_alignment(dtype, V, B, rule):
    """TV slices as job-pass items: per-sequence rules."""
    assert route(B, 1, V, dtype, rule, per_seq=True) & TV_JOBS
    wl = W.WORKLOADS[3].with_(B=B, gamma=1, V=V, dtype=dtype, rule=rule, alpha=0.1)
    check(W.generate(wl, 33, DEV), dtype, per_seq=True)


@pytest.mark.parametrize("B,dtype,V,rule,path", [
    (100, "bf16", 1001, W.OPT, SEQ), (16, "bf16", 1001, W.TOKEN_V2, SEQ),
    (16, "bf16", 1001, W.DIFFLOG, SEQ), (100, "f32", 1001, W.OPT, SEQ),
    (16, "f32", 1001, W.TOKEN_V2, SEQ), (16, "f32", 1001, W.DIFFLOG, SEQ),
    (16, "bf16", 1001, W.OPT, SMALL), (16, "bf16", 20003, W.OPT, SMALL),
    (16, "bf16", 20003, W.TOKEN_V2, SMALL), (16, "bf16", 9003, W.DIFFLOG, SMALL),
    (16, "f32", 9999, W.OPT, SMALL), (16, "f32", 9999, W.TOKEN_V2, SMALL),
    (16, "f32", 9999, W.DIFFLOG, SMALL), (16, "bf16", 40003, W.OPT, TILES),
    (16, "bf16", 40003, W.TOKEN_V2, TILES), (16, "bf16", 20003, W.DIFFLOG, TILES),
    (16, "bf16", 40003, W.DIFFLOG, TILES), (16, "f32", 20001, W.OPT, TILES),
    (16, "f32", 20001, W.TOKEN_V2, TILES), (16, "f32", 20001, W.DIFFLOG, TILES)])
def test_rows_do_not_depend_on_their_alignment(B, dtype, V, rule, path):
    """The same row at every position of the batch, so at every alignment,
    gives bitwise the same statistics and the same draw."""
    g1 = 3
    assert route(B, g1 - 1, V, dtype, rule) & path
    g = torch.Generator(device=DEV).manual_seed(3)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    row = torch.randn(2, V, generator=g, device=DEV).to(dt)
    q, p = (row[i].expand(B, g1, V).contiguous() for i in range(2))
    draft = torch.zeros(B, g1 - 1, dtype=torch.int32, device=DEV)
    st = torch.empty(B, g1, 8, device=DEV)
    norm = torch.empty(B, device=DEV)
    u = torch.full((B, g1), 0.5, device=DEV)
    _, tok, _ = spc.spc_verify_ex(q, p, draft, u, rule, 0.1, 1.0, out_row_stats=st,
                                  out_sample_norm=norm)
    # (a token rule's row reports r at its own draft; the draft is the same)
    assert torch.equal(st, st[:1, :1].expand(B, g1, 8))
    assert torch.equal(tok, tok[:1].expand(B))
    assert torch.equal(norm, norm[:1].expand(B))


# A workgroup per sequence: one to sixteen wavefronts a row, more rows than
# wavefronts, one to four lane loads at a time, and rows that end inside a
# lane load.  (A shape whose rule makes it longer than this path takes runs
# on the next one.)
@pytest.mark.parametrize("dtype,B,gamma,V", [
    ("bf16", 3, 1, 2), ("f32", 3, 1, 3), ("bf16", 5, 15, 255), ("f32", 4, 16, 239),
    ("bf16", 2, 63, 64), ("f32", 3, 2, 1365), ("bf16", 7, 7, 513), ("bf16", 3, 1, 4096),
    ("f32", 3, 1, 2047), ("bf16", 300, 4, 1025), ("f32", 140, 4, 4095), ("bf16", 65, 7, 2559),
    ("f32", 129, 1, 10239)])
@pytest.mark.parametrize("rule", [W.DIFF, W.OPT, W.TOKEN_V2, W.LOSSY, W.BILD, W.OPTLOG])
@pytest.mark.parametrize("greedy", [False, True])
def test_short_sequences(dtype, B, gamma, V, rule, greedy):
    wl = W.WORKLOADS[3].with_(B=B, gamma=gamma, V=V, dtype=dtype, rule=rule, alpha=0.1,
                              temperature=0.0 if greedy else 0.7)
    inp = W.generate(wl, 57, DEV)
    with_stats = check(inp, dtype, greedy)
    plain = check(inp, dtype, greedy, stats=False)
    for k in ("accept_len", "next_token", "defer"):
        np.testing.assert_array_equal(plain[k], with_stats[k])


# The longest sequences that path takes.
@pytest.mark.parametrize("dtype,B,gamma,V,rule", [
    ("bf16", 3, 1, 4095, W.DIFF), ("f32", 3, 3, 1023, W.LOSSY), ("bf16", 3, 1, 1023, W.OPT),
    ("bf16", 3, 1, 3071, W.DIFFLOG), ("f32", 3, 1, 2303, W.DIFFLOG),
    ("f32", 129, 1, 8191, W.DIFFLOG), ("bf16", 129, 1, 16383, W.DIFFLOG),
    ("bf16", 513, 6, 2047, W.DIFF), ("f32", 513, 6, 1023, W.OPT), ("bf16", 513, 5, 6399, W.TOKEN_V2),
    ("f32", 2, 3, 1023, W.TOKEN_V1), ("bf16", 4, 3, 1021, W.TOKEN_V3),
    ("bf16", 129, 1, 20479, W.DIFF), ("f32", 129, 1, 20479, W.LOSSY),
    ("f32", 60, 4, 8191, W.TOKEN_V2), ("bf16", 129, 1, 20477, W.TOKEN_V1),
    ("bf16", 129, 1, 10239, W.OPT), ("f32", 60, 4, 4095, W.OPT)])
def test_longest_short_sequences(dtype, B, gamma, V, rule):
    assert route(B, gamma, V, dtype, rule) & SEQ
    wl = W.WORKLOADS[3].with_(B=B, gamma=gamma, V=V, dtype=dtype, rule=rule, alpha=0.1)
    inp = W.generate(wl, 58, DEV)
    check(inp, dtype)
    check(inp, dtype, stats=False)


@pytest.mark.parametrize("B,dtype,gamma,V", [
    (8, "bf16", 2, 1201), (8, "f32", 4, 810), (8, "bf16", 3, 1000), (100, "bf16", 2, 1201),
    (100, "f32", 4, 810), (100, "bf16", 3, 1000), (8, "bf16", 2, 9001), (8, "f32", 4, 8100)])
@pytest.mark.parametrize("rule,alpha", [(W.OPT, 0.1), (W.TOKEN_V2, 0.05), (W.BILD, 6.0),
                                        (W.OPTLOG, 1.0), (W.LOSSY, 0.3)])
def test_short_sequences_masked(B, dtype, gamma, V, rule, alpha):
    """-inf entries in both tensors, whole lane loads and wavefronts among
    them: a workgroup per sequence, or (few long rows) per row."""
    assert route(B, gamma, V, dtype, rule) & (SEQ if B == 100 else SMALL if V > 8000 else
                                              SEQ | SMALL)
    wl = W.WORKLOADS[3].with_(B=B, gamma=gamma, V=V, dtype=dtype, rule=rule, alpha=alpha)
    inp = W.generate(wl, 2, DEV)
    g0 = torch.Generator(device=DEV).manual_seed(99)
    for k in ("q", "p"):
        m = torch.rand(inp[k].shape, generator=g0, device=DEV) < 0.3
        m[1::3, :, 128:700] = True
        m[..., 0] = False  # at least one finite entry per row
        if k == "p" and rule == W.BILD:
            m[::2] = False  # half the sequences keep a finite cross-entropy
        inp[k][m] = float("-inf")
    inp["draft"] = W.draw_drafts(inp["q"], inp["temperature"], g0)
    check(inp, dtype)


@pytest.mark.parametrize("B,dtype,gamma,V,path", [
    (8, "bf16", 2, 1201, SEQ), (8, "f32", 3, 1021, SEQ), (150, "bf16", 1, 3000, SEQ),
    (70, "f32", 4, 1023, SEQ), (70, "f32", 4, 1203, TILES), (8, "f32", 4, 1203, SMALL), (8, "bf16", 1, 3000, SMALL),
    (8, "bf16", 4, 8191, SMALL)])
def test_short_sequences_argmax_ties(B, dtype, gamma, V, path):
    """Ties within a lane load, across lanes, lane loads and wavefronts: the
    lowest index, batch-wide and per sequence."""
    assert route(B, gamma, V, dtype, W.OPT, greedy=True) & path
    wl = W.WORKLOADS[4].with_(B=B, gamma=gamma, V=V, dtype=dtype)
    inp = W.generate(wl, 9, DEV)
    rng = np.random.default_rng(4)
    low = {}
    for k in ("q", "p"):
        x = inp[k].float().cpu().numpy()
        low[k] = np.empty(x.shape[:2], np.int64)
        for i in np.ndindex(*x.shape[:2]):
            n = int(rng.integers(0, V - 530))
            pos = ([V - 1, V - 2, 0], [n + 3, n + 1], [n + 512, n + 9, n + 64],
                   list(rng.choice(V, 9, replace=False)), [V - 1, V - 3])[int(rng.integers(0, 5))]
            x[i][pos] = float(np.ceil(x[i].max())) + 1.0
            low[k][i] = min(pos)
        inp[k].copy_(torch.from_numpy(x).to(inp[k].dtype))
    g = check(inp, dtype, greedy=True)
    for c, k in enumerate(("q", "p")):
        np.testing.assert_array_equal(g["argmax"][..., c], low[k])
    check(inp, dtype, greedy=True, per_seq=True)


# Rows held by a workgroup, with and without first moments: the shortest and
# longest of their range, a whole number of lane loads and an entry either side.
@pytest.mark.parametrize("dtype,B,gamma,V", [
    ("bf16", 6, 7, 1999), ("bf16", 6, 7, 2048), ("bf16", 6, 7, 8191), ("bf16", 6, 7, 8193),
    ("bf16", 5, 3, 16383), ("bf16", 5, 3, 16384), ("f32", 6, 7, 1021), ("f32", 6, 7, 4095),
    ("f32", 6, 7, 4096), ("f32", 6, 7, 4097), ("f32", 5, 3, 16383), ("f32", 5, 3, 16384)])
@pytest.mark.parametrize("rule,alpha,greedy", [
    (W.OPT, 0.1, False), (W.DIFFLOG, 0.5, False), (W.OPTLOG, 0.5, False), (W.BILD, 1.0, False),
    (W.TOKEN_V1, 0.1, False), (W.DIFFLOG, 0.5, True), (W.OPT, 0.1, True)])
def test_rows_held_by_a_workgroup(dtype, B, gamma, V, rule, alpha, greedy):
    assert route(B, gamma, V, dtype, rule, greedy) & SMALL or (
        greedy and (V > 8192 or rule == W.OPT))
    wl = W.WORKLOADS[3].with_(B=B, gamma=gamma, V=V, dtype=dtype, rule=rule, alpha=alpha,
                              temperature=0.0 if greedy else 0.8)
    inp = W.generate(wl, 59, DEV)
    with_stats = check(inp, dtype, greedy)
    plain = check(inp, dtype, greedy, stats=False)
    for k in ("accept_len", "next_token", "defer"):
        np.testing.assert_array_equal(plain[k], with_stats[k])


@pytest.mark.parametrize("dtype,gamma,V", [("bf16", 3, 1001), ("f32", 4, 800), ("bf16", 6, 1170),
                                           ("bf16", 1, 16001), ("f32", 2, 12000)])
def test_short_sequences_identical_models(dtype, gamma, V):
    """p = q: every draft is kept, D_TV and H(q) - H(p) are exactly 0."""
    wl = W.WORKLOADS[3].with_(B=9, gamma=gamma, V=V, dtype=dtype)
    same = W.generate(wl, 3, DEV)
    same["p"] = same["q"].clone()
    for rule, alpha in ((W.LOSSY, 0.3), (W.DIFFLOG, 0.0), (W.OPTLOG, 0.5), (W.DIFF, 0.0),
                        (W.OPT, 0.1)):
        same["rule"][:] = rule
        same["alpha"][:] = alpha
        g = check(same, dtype)
        assert (g["accept_len"] == gamma).all() and (g["defer"] == 0).all()
        if rule in (W.OPT, W.OPTLOG):
            assert (g["row_stats"][..., 6] == 0).all()
        if rule in (W.DIFFLOG, W.OPTLOG):
            assert (g["row_stats"][..., 7] == 0).all()


# TV passes from the rows' own tiles, either side of the most tiles a row's
# gate holds (62 of 4096 float32 entries), with the wait as it is and at 0
# ticks (every workgroup that does not find its row merged leaves its tile to
# the merge), with row statistics (every row takes its TV pass) and without
# (rows D_TV cannot change are decided at their merge and skip theirs).
@pytest.mark.parametrize("ticks", [None, "0"])
@pytest.mark.parametrize("dtype,B,gamma,V,rule,want", [
    ("f32", 1, 2, 253952, W.OPT, TV_SELF), ("f32", 1, 2, 253953, W.OPT, TV_PASS),
    ("f32", 1, 1, 253952, W.OPTLOG, TV_SELF), ("f32", 1, 1, 256000, W.OPTLOG, TV_PASS), ("f32", 8, 5, 32128, W.OPT, TV_SELF),
    ("bf16", 4, 2, 100003, W.OPT, TV_SELF), ("bf16", 4, 2, 100003, W.OPTLOG, TV_SELF)])
def test_tv_pass_from_resident_tiles(dtype, B, gamma, V, rule, want, ticks, monkeypatch):
    if ticks is not None:
        monkeypatch.setenv("SPC_TV_WAIT_TICKS", ticks)
    assert route(B, gamma, V, dtype, rule) & want
    wl = W.WORKLOADS[3].with_(B=B, gamma=gamma, V=V, dtype=dtype, rule=rule,
                              alpha=0.1 if rule == W.OPT else 0.5)
    for step in (21, 22, 23):
        inp = W.generate(wl, step, DEV)
        check(inp, dtype)
        check(inp, dtype, stats=False)


@pytest.mark.parametrize("dtype,B,gamma,V", [("bf16", 12, 4, 800), ("f32", 90, 3, 4000), ("f32", 12, 3, 5001),
                                             ("bf16", 12, 3, 12000), ("f32", 90, 3, 5000)])
def test_short_sequences_mixed(dtype, B, gamma, V):
    """Per-sequence rules and temperatures, and an out-of-range draft."""
    wl = W.WORKLOADS[5].with_(B=B, gamma=gamma, V=V, dtype=dtype)
    inp = W.generate(wl, 3, DEV)
    g = torch.Generator(device=DEV).manual_seed(1)
    inp["rule"] = torch.randint(0, 13, (B,), generator=g, device=DEV, dtype=torch.int32)
    inp["draft"][1] = V + 3
    a = parity.run_gpu(inp, per_seq=True)
    h = parity.host_inputs(inp)
    parity.compare(a, parity.run_oracle(h), h, dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V", [3, 4096, 4097, 8192, 8193, 64 * 8192 + 5, 65 * 4096])
@pytest.mark.parametrize("T", [1.0, 0.0])
def test_drafter_rows_of_one_tile_and_of_many(dtype, V, T):
    """One tile (nothing published), two, and either side of a tile per lane."""
    wl = W.WORKLOADS[3].with_(B=9, V=V, dtype=dtype)
    z = W.generate(wl, 6, DEV)["q"][:, 0].contiguous()
    u = torch.rand(9, generator=torch.Generator(device=DEV).manual_seed(2), device=DEV)
    tok = spc.spc_draft_sample(z, T, uniforms=u).cpu().numpy()
    o_tok, o_margin = oracle.draft_sample(parity.host_logits(z), np.full(9, T, np.float32),
                                          u.cpu().numpy())
    for g, o, m in zip(tok, o_tok, o_margin):
        assert g == o or m < parity.NEAR, (g, o, m)


# The mean (rms) error of a row's largest probability against float64.  Its
# own float32 rounding and the hardware exponentials leave 1.6e-8 to 2.2e-8 on
# every path.  With references moved by an uncorrected float32 exponential
# (short sequences) or a thread's whole share summed in float32 it was 2.8e-8
# to 3.2e-8; the bound lies between.
@pytest.mark.parametrize("dtype,V,path", [
    ("bf16", 1001, SEQ), ("f32", 1001, SEQ), ("f32", 2001, SMALL), ("bf16", 2083, SMALL),
    ("bf16", 20003, SMALL), ("bf16", 60003, TILES), ("bf16", 100003, TILES),
    ("f32", 60003, TILES)])
@pytest.mark.parametrize("moments", [False, True])
def test_rounding_of_the_largest_probability(dtype, V, path, moments):
    B, gamma, T = 24, 7, 0.7
    if moments:
        if path == SMALL:
            V = min(V, 16001)
        elif path == SEQ:
            B = 50
    rule = (W.OPTLOG if path & TILES else W.DIFFLOG) if moments else W.OPT if path & TILES else W.CHOW
    assert route(B, gamma, V, dtype, rule) & path
    d2, n = 0.0, 0
    for step in range(4):
        wl = W.WORKLOADS[3].with_(B=B, gamma=gamma, V=V, dtype=dtype, rule=rule, temperature=T)
        inp = W.generate(wl, 900 + step, DEV)
        st = torch.empty(B, gamma + 1, 8, device=DEV)
        spc.spc_verify_ex(inp["q"], inp["p"], inp["draft"], inp["uniforms"], rule, 0.1, T,
                          out_row_stats=st)
        for c, k in ((2, "q"), (5, "p")):
            z = inp[k].double() / float(np.float32(T))
            d = st[..., c].double() - (z.max(-1).values - z.logsumexp(-1)).exp()
            d2, n = d2 + float(d.pow(2).sum()), n + d.numel()
    assert (d2 / n) ** 0.5 < 2.6e-8


# The mass reported for a draw from q, p or a token rule's target: these sum to
# 1 by the row's normalisers, which the value reported must show to a unit in
# the last place below 1 (summing the float32 weights that the search uses
# leaves errors of 1.2e-7 to 7e-7).
@pytest.mark.parametrize("dtype,B,V,path", [
    ("bf16", 100, 1001, SEQ), ("f32", 100, 1000, SEQ), ("bf16", 40, 3001, SMALL),
    ("f32", 40, 4096, SMALL), ("bf16", 24, 16001, SMALL), ("bf16", 24, 60003, TILES)])
@pytest.mark.parametrize("rule", [W.OPT, W.TOKEN_V2, W.DIFFLOG])
def test_mass_of_an_extra_token_draw(dtype, B, V, path, rule):
    gamma = 2
    assert route(B, gamma, V, dtype, rule) & path
    seen = 0
    for step in range(4):
        wl = W.WORKLOADS[3].with_(B=B, gamma=gamma, V=V, dtype=dtype, rule=rule, alpha=0.1)
        inp = W.generate(wl, 700 + step, DEV)
        if rule != W.TOKEN_V2:
            inp["p"] = inp["q"].clone()  # every draft is kept
        norm = torch.empty(B, device=DEV)
        acc, _, _ = spc.spc_verify_ex(inp["q"], inp["p"], inp["draft"], inp["uniforms"], rule, 0.1,
                                      1.0, out_sample_norm=norm)
        w = norm[acc == gamma]
        seen += w.numel()
        # (a token rule's target as tiles: eta's own rounding)
        bound = 2.5e-7 if path == TILES and rule == W.TOKEN_V2 else 6e-8
        assert ((w - 1).abs() <= bound).all(), (w - 1).abs().max()
    assert seen


# The mean error of eta against float64: rows at any alignment held by a
# workgroup are no worse than statistics tiles (2.9e-8; from the marked mass
# alone 4.2e-8 to 5.0e-8).
@pytest.mark.parametrize("dtype,V", [("bf16", 10007), ("bf16", 20003), ("f32", 10007)])
def test_rounding_of_eta(dtype, V):
    B, gamma, alpha, T = 12, 5, 0.1, 0.7
    assert route(B, gamma, V, dtype, W.TOKEN_V2) & SMALL
    d2, n = 0.0, 0
    for step in range(12):
        wl = W.WORKLOADS[3].with_(B=B, gamma=gamma, V=V, dtype=dtype, rule=W.TOKEN_V2, alpha=alpha,
                                  temperature=T)
        inp = W.generate(wl, 800 + step, DEV)
        st = torch.empty(B, gamma + 1, 8, device=DEV)
        spc.spc_verify_ex(inp["q"], inp["p"], inp["draft"], inp["uniforms"], W.TOKEN_V2, alpha, T,
                          out_row_stats=st)
        q, p = ((inp[k].double() / float(np.float32(T))).softmax(-1) for k in "qp")
        r = p < p.max(-1, keepdim=True).values - float(np.float32(alpha))
        d = st[..., 6].double() - (q * r).sum(-1)
        d = d[d.abs() < 1e-6]  # (a near-tie of r moves eta by its entry)
        d2, n = d2 + float(d.pow(2).sum()), n + d.numel()
    assert n > 0.97 * 12 * B * (gamma + 1)
    assert (d2 / n) ** 0.5 < 3.6e-8
