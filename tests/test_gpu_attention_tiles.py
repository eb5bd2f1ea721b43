"""Group attention at the sizes where the tiles change, through the C ABI:
128-query tasks (long sequences) and each tile size of the projections, on
sampled query rows against the per-row oracle."""

import numpy as np
import pytest

from oracle import attention_oracle as ao
from paper_2605_06206_amd import synth
from test_gpu_attention import TOL, _run, attn_part_err, rel_err, say

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
