"""The grouped expert FFN at the edges of its tiles, through the C ABI: row
counts around the tile rows and their halves, K and N remainders, and odd
numbers of K stages.  Workspace and output start as NaN, so a row or column
read from outside its operand shows."""

import numpy as np
import pytest
import torch

from oracle import foe_oracle as oracle
from paper_2605_06206_amd import foe, synth

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


DT = {"bf16": (torch.bfloat16, foe.BF16), "f32": (torch.float32, foe.F32)}
# largest error over the largest value of an expert.  bf16: h and y are rounded
# (2^-9 each, relative) and cancel in the sums; fp32: sums of up to 520
# products, 2^-24 each
TOL = {"bf16": 2e-2, "f32": 1e-5}


def _poison(shape, dtype):
    n = int(np.prod(shape)) * torch.empty(0, dtype=dtype).element_size()
    return torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda").view(dtype).view(shape)


# rows per expert; every list averages at least 64 rows (the tiled kernels)
ROWS = {
    "tile edges": [255, 256, 257, 0, 1],
    "half tile edges": [127, 128, 129, 384, 385],
    "16-row edges": [15, 16, 17, 400, 63],
    "one expert": [1000],
    "many small, one large": [3, 0, 70, 700, 5, 64],
}
# (d, F): K stages of 64 columns, so d = 72 is two stages with a remainder of
# 8, 192 an odd number of stages, and 8 less than one stage
WIDTHS = [(256, 192), (72, 136), (192, 64), (8, 328), (520, 72)]


@pytest.mark.parametrize("rows", list(ROWS))
@pytest.mark.parametrize("d,F", WIDTHS)
@pytest.mark.parametrize("dt", list(DT))
def test_expert_ffn_tile_edges(rows, d, F, dt):
    counts = ROWS[rows]
    E, R = len(counts), sum(counts)
    print("expert_ffn edges", rows, d, F, dt, flush=True)
    dtype, code = DT[dt]
    inp = synth.make_ffn_inputs(R, E, d, F, seed=R + d, sigma=0.05, dtype=dt)
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    ws = _poison((foe.workspace_bytes("expert_ffn", code, 1, R, d, E, 1, F),), torch.uint8)
    x, wg, wu, wd = (_dev(inp[n]).to(dtype) for n in ("x_perm", "w_gate", "w_up", "w_down"))
    y = foe.expert_ffn(x, _dev(off), wg, wu, wd, y_perm=_poison((R, d), dtype), ws=ws)
    got = y.float().cpu().numpy()
    ref = oracle.expert_ffn(inp["x_perm"], off, inp["w_gate"], inp["w_up"], inp["w_down"])
    assert np.isfinite(got).all()
    for e in range(E):
        a, b = off[e], off[e + 1]
        if b > a:
            err = np.abs(got[a:b] - ref[a:b]).max() / np.abs(ref[a:b]).max()
            assert err <= TOL[dt], (rows, e, err)
