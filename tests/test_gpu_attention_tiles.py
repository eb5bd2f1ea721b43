"""Group attention at the sizes where the tiles change, through the C ABI:
128-query tasks (long sequences) and each tile size of the projections, on
sampled query rows against the per-row oracle."""

import numpy as np
import pytest
import torch

from oracle import attention_oracle as ao
from paper_2605_06206_amd import foe, synth
from test_gpu_attention import TOL, _check, _run, attn_part_err, rel_err, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,S,d,nq,hd", [
    (8, 2945, 72, 4, 128),   # 24 x 16 tasks of 128 queries, two heads each; last block of 1 row
    (8, 3072, 72, 4, 96),    # whole tasks; V^T loads uneven over the waves
    (8, 1700, 72, 3, 128),   # one head per task, two key parts
    (8, 1729, 104, 3, 96),
    (8, 2944, 72, 4, 128),   # one task fewer: 64 queries
    (4, 1025, 1032, 2, 128),  # projections: 128 x 128 and 64 x 128 tiles
    (2, 1500, 1544, 2, 128),  # output projection: 128 x 128 tiles
])
def test_group_attention_tile_forms(H, S, d, nq, hd):
    cfg = dict(H=H, S=S, d=d, nq=nq, hd=hd, theta=10000.0, scale=1.0, sigma=0.05, seed=S + d)
    say("tile forms", cfg)
    inp = synth.make_attention_inputs(cfg)
    got = _run(inp)
    assert np.isfinite(got).all()
    edges = [0, 1, 31, 32, 63, 64, 127, 128, 129, S // 2, S - 130, S - 65, S - 2, S - 1]
    rows = sorted({r for r in edges if 0 <= r < S})
    x = inp["x"].astype(np.float64)
    ref = np.zeros((len(rows), d))
    for h, g in enumerate(inp["groups"]):
        ref += x[h, rows] + ao.group_attention_rows(x[h], g["w_qkv"], g["w_o"], nq, hd, 10000.0,
                                                    1.0, rows)
    ref /= H
    e_full, e_attn = rel_err(got[rows], ref), attn_part_err(got[rows], ref, x[:, rows].mean(axis=0))
    say(f"rel err r_full {e_full:.2e}, attention part {e_attn:.2e}")
    assert e_full <= TOL and e_attn <= TOL


@pytest.mark.parametrize("S", [300, 312])
def test_group_attention_capture_with_and_without_side_stream(S):
    """The residual sum of 300 rows (49.2 MB of x) runs in the preparation
    launch, that of 312 (51.1 MB) on the side stream, forked and joined inside
    the capture: replays give the eager bits, with the workspace poisoned in
    between, and the residual alone (zero projections) is the mean over groups."""
    H, d, nq, hd = 8, 10240, 1, 96
    say("capture", S)
    gen = torch.Generator(device="cuda").manual_seed(S)
    x = torch.randn((H, S, d), generator=gen, device="cuda").to(torch.bfloat16)
    wq = (torch.randn((H, (nq + 2) * hd, d), generator=gen, device="cuda") * 0.01).to(torch.bfloat16)
    wo = (torch.randn((d, H * nq * hd), generator=gen, device="cuda") * 0.03).to(torch.bfloat16)
    n = foe.lib().foe_group_attention_workspace_bytes(H, S, d, nq, hd)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    out = torch.empty((S, d), dtype=torch.bfloat16, device="cuda")
    mean = foe.group_attention(x, wq, torch.zeros_like(wo), nq, 1e4, 1.0, ws=ws).float()
    ref = x.double().mean(0)
    # one rounding to bf16 of sums that are exact to 2^-24
    assert ((mean - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-6).all()
    eager = foe.group_attention(x, wq, wo, nq, 1e4, 1.0, ws=ws).clone()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        foe.group_attention(x, wq, wo, nq, 1e4, 1.0, out=out, ws=ws)
    for _ in range(3):
        ws.fill_(255)
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager)


@pytest.mark.parametrize("H,S,d,nq,hd", [
    (64, 700, 64, 2, 128), (64, 700, 64, 2, 96),   # 128-query tasks, one and two key parts
    (64, 700, 64, 1, 128), (64, 700, 64, 1, 96),
    (2, 700, 64, 2, 128), (2, 700, 64, 1, 96),     # 64-query tasks
])
@pytest.mark.parametrize("t", [64, 192, 640])
def test_tokens_before_a_non_finite_one_keep_their_bits(H, S, d, nq, hd, t):
    """A token whose x is infinite makes its k and v non-finite; the rows before
    it (in 64-key blocks before its own) never see them."""
    say("non-finite token", (H, S, d, nq, hd, t))
    gen = torch.Generator(device="cuda").manual_seed(t)
    x = torch.randn((H, S, d), generator=gen, device="cuda").to(torch.bfloat16)
    wq = (torch.randn((H, (nq + 2) * hd, d), generator=gen, device="cuda") * 0.1).to(torch.bfloat16)
    wo = (torch.randn((d, H * nq * hd), generator=gen, device="cuda") * 0.03).to(torch.bfloat16)
    ref = foe.group_attention(x, wq, wo, nq, 1e4, 1.0).clone()
    assert torch.isfinite(ref.float()).all()
    x[0, t] = float("inf")
    got = foe.group_attention(x, wq, wo, nq, 1e4, 1.0)
    assert torch.equal(got[:t], ref[:t])
    assert torch.isnan(got[t].float()).all()


@pytest.mark.parametrize("theta", [3e38, float("inf")])
def test_largest_rotary_bases(theta):
    """The rotary base may be any positive float: with an infinite one the first
    pair of a head rotates by the position and the others stay."""
    say("rotary base", theta)
    inp = synth.make_attention_inputs(dict(H=2, S=40, d=64, nq=2, hd=128, theta=theta, scale=1.0,
                                           sigma=0.05, seed=3))
    got = _run(inp)
    assert np.isfinite(got).all()
    _check(inp, got)
