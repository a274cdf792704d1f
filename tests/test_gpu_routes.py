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


# Rows that start inside a 16-byte vector and end inside a lane load: fewer
# entries than one vector, one entry either side of a vector, of a
# wavefront's lane load and of a tile (8192 bfloat16 / 4096 float32), on the
# statistics-tile path (more rows than the one-launch paths take).
@pytest.mark.parametrize("dtype,V,B,rule", [
    ("bf16", 2, 300, W.DIFF), ("bf16", 7, 300, W.OPT), ("bf16", 9, 300, W.TOKEN_V2),
    ("bf16", 511, 300, W.LOSSY), ("bf16", 513, 300, W.OPT), ("bf16", 8191, 280, W.DIFF),
    ("bf16", 8193, 280, W.TOKEN_V1), ("bf16", 40001, 5, W.OPT), ("bf16", 65543, 70, W.DIFF),
    ("f32", 3, 300, W.DIFF), ("f32", 5, 300, W.OPT), ("f32", 4095, 280, W.BILD),
    ("f32", 4097, 280, W.DIFFLOG), ("f32", 33333, 6, W.OPTLOG)])
@pytest.mark.parametrize("greedy", [False, True])
def test_rows_at_any_alignment(dtype, V, B, rule, greedy):
    wl = W.WORKLOADS[3].with_(B=B, gamma=1, V=V, dtype=dtype, rule=rule, alpha=0.1,
                              temperature=0.0 if greedy else 1.0)
    parity.parity_workload(wl, 1, step0=31, report_name=f"anyalign.{dtype}.{V}")


@pytest.mark.parametrize("dtype,V", [("bf16", 20003), ("f32", 9999)])
def test_rows_do_not_depend_on_their_alignment(dtype, V):
    """The same row at every position of the batch, so at every alignment,
    gives bitwise the same statistics."""
    g = torch.Generator(device=DEV).manual_seed(3)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    B, g1 = 16, 3
    row = torch.randn(2, V, generator=g, device=DEV).to(dt)
    q, p = (row[i].expand(B, g1, V).contiguous() for i in range(2))
    draft = torch.zeros(B, g1 - 1, dtype=torch.int32, device=DEV)
    st = torch.empty(B, g1, 8, device=DEV)
    u = torch.full((B, g1), 0.5, device=DEV)
    _, tok, _ = spc.spc_verify_ex(q, p, draft, u, W.OPT, 0.1, 1.0, out_row_stats=st)
    assert torch.equal(st, st[:1, :1].expand(B, g1, 8))
    assert torch.equal(tok, tok[:1].expand(B))


# A workgroup per sequence: one to sixteen wavefronts a row, more rows than
# wavefronts, one to four lane loads at a time, rows that end inside a lane
# load, and the longest sequences it takes (few rows: 8192 entries, 4096 with
# a second pass; many: 40960, 20480).
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
    parity.parity_workload(wl, 1, step0=57, stats=V % 2 == 0, report_name=f"seq.{dtype}.{V}")


@pytest.mark.parametrize("dtype,B,gamma,V", [("bf16", 12, 4, 800), ("f32", 90, 3, 5000)])
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
