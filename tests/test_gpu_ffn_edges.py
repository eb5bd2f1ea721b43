"""The grouped expert FFN at the edges of its tiles and of the rule that picks
them, through the C ABI: row counts around the tile rows and their halves, K
and N remainders, and odd numbers of K stages.  Workspace and output start as
NaN, so a row or column read from outside its operand shows."""

import numpy as np
import pytest
import torch

import block_check as bc
from oracle import foe_oracle as oracle
from paper_2605_06206_amd import foe, synth

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


DT = {"bf16": (torch.bfloat16, foe.BF16), "f32": (torch.float32, foe.F32)}
# largest error over the largest value of an expert.  bf16: h and y are rounded
# (2^-9 each, relative) and cancel in the sums; fp32: sums of up to 8320
# products, each term within 2^-24 of the running sum
TOL = {"bf16": 2e-2, "f32": 1e-5}


def _poison(shape, dtype):
    n = int(np.prod(shape)) * torch.empty(0, dtype=dtype).element_size()
    return torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda").view(dtype).view(shape)


# rows per expert; every list averages at least 32 rows (the tiled kernels)
ROWS = {
    "tile edges": [255, 256, 257, 0, 1],
    "half tile edges": [127, 128, 129, 384, 385],
    "16-row edges": [15, 16, 17, 400, 63],
    "one expert": [1000],
    "many small, one large": [3, 0, 70, 700, 5, 64],
    "medium tiles": [64, 65, 32, 33, 0, 31],
}
# (d, F): K stages of 64 columns, so d = 72 is two stages with a remainder of
# 8, 192 an odd number of stages, and 8 less than one stage; the wide F of the
# last two makes enough tiles for the large ones (from 96 rows per expert on)
WIDTHS = [(256, 192), (72, 136), (192, 64), (8, 328), (520, 72), (72, 8008), (192, 8320)]


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


@pytest.mark.parametrize("T,d,E,k,F", [
    (31, 64, 2, 2, 64),     # 31 and 32 rows per expert: weight stream, medium tiles
    (32, 64, 2, 2, 64),
    (95, 64, 2, 2, 64),     # below 96 rows: medium tiles whatever the width
    (700, 72, 4, 2, 4416),  # both GEMMs in one launch, d off the tile, odd K stages
    (513, 192, 2, 1, 8384),
    (700, 72, 4, 2, 4424),  # as two launches of large tiles (F not a multiple of 64)
])
def test_block_ffn_forms(T, d, E, k, F):
    """The block on both sides of the FFN's form rule; every expert row of the
    update (the output without the residual) against the oracle."""
    print("block ffn forms", T, d, E, k, F, flush=True)
    inp = synth.make_block_inputs(dict(dtype="bf16", C=1, T=T, d=d, E=E, k=k, F=F, sigma=0.05,
                                       seed=T + d, bias=None))
    cl = inp["clusters"][0]
    routes = bc.oracle_routes(inp["x"], inp["clusters"], k)
    assert not bc.exempt_mask(routes).any()
    ref, _, _ = bc.oracle_block(inp["x"], inp["clusters"], k, None, "renorm", routes=routes)
    x, wr, wg, wu, wd = (_dev(a).to(torch.bfloat16) for a in (
        inp["x"], cl["w_router"], cl["w_gate"], cl["w_up"], cl["w_down"]))
    ws = _poison((foe.workspace_bytes("cluster_block", foe.BF16, 1, T, d, E, k, F),), torch.uint8)
    got = foe.cluster_block(x, wr[None], None, wg[None], wu[None], wd[None], k, ws=ws,
                            out=_poison((T, d), torch.bfloat16)).float().cpu().numpy()
    assert np.isfinite(got).all()
    e_out, e_upd = bc.block_errors(got, ref, inp["x"], 1, None, "bf16")
    assert e_out <= bc.TOL["bf16"] and e_upd <= bc.TOL["bf16"], (e_out, e_upd)


@pytest.mark.parametrize("T,d,E,k,F,C", [
    (1, 64, 8, 2, 64, 3),     # two pairs per cluster
    (5, 72, 32, 4, 136, 2),   # 20 pairs, some experts several times
    (32, 64, 64, 2, 64, 1),   # 64 pairs: the most that one wave lists
    (33, 64, 64, 2, 64, 1),   # one token more
    (3, 64, 100, 1, 64, 2),   # three pairs among 100 experts
    (11, 64, 8, 1, 64, 1),    # 11 and 12 pairs for 8 experts: both sides of the rule
    (12, 64, 8, 1, 64, 1),
])
def test_block_few_pairs(T, d, E, k, F, C):
    """Few pairs per cluster: workgroups numbered by distinct expert."""
    print("block few pairs", T, d, E, k, F, C, flush=True)
    inp = synth.make_block_inputs(dict(dtype="bf16", C=C, T=T, d=d, E=E, k=k, F=F, sigma=0.05,
                                       seed=7 * T + d, bias=None))
    routes = bc.oracle_routes(inp["x"], inp["clusters"], k)
    assert not bc.exempt_mask(routes).any()
    ref, _, _ = bc.oracle_block(inp["x"], inp["clusters"], k, None, "renorm", routes=routes)
    w = {n: _dev(np.stack([cl[n] for cl in inp["clusters"]])).to(torch.bfloat16)
         for n in ("w_router", "w_gate", "w_up", "w_down")}
    ws = _poison((foe.workspace_bytes("cluster_block", foe.BF16, C, T, d, E, k, F),), torch.uint8)
    got = foe.cluster_block(_dev(inp["x"]).to(torch.bfloat16), w["w_router"], None, w["w_gate"],
                            w["w_up"], w["w_down"], k, ws=ws,
                            out=_poison((T, d), torch.bfloat16)).float().cpu().numpy()
    assert np.isfinite(got).all()
    e_out, e_upd = bc.block_errors(got, ref, inp["x"], C, None, "bf16")
    assert e_out <= bc.TOL["bf16"] and e_upd <= bc.TOL["bf16"], (e_out, e_upd)


@pytest.mark.parametrize("T,E,k,C", [
    (1, 8, 2, 2),     # workgroups by distinct expert
    (7, 8, 2, 1),
    (20, 8, 1, 4),    # workgroups by expert
    (100, 8, 2, 2),   # through the index pass or the stream's parts
    (300, 4, 2, 1),
    (700, 2, 2, 1),   # tiles
])
def test_block_token_without_an_expert(T, E, k, C):
    """A token with a NaN selects no expert (its scores are NaN): its output row is
    the residual in every form, and the other rows do not change."""
    print("block NaN token", T, E, k, C, flush=True)
    d, F = 72, 64
    inp = synth.make_block_inputs(dict(dtype="bf16", C=C, T=T, d=d, E=E, k=k, F=F, sigma=0.05,
                                       seed=T, bias=None))
    w = {n: _dev(np.stack([cl[n] for cl in inp["clusters"]])).to(torch.bfloat16)
         for n in ("w_router", "w_gate", "w_up", "w_down")}
    x = _dev(inp["x"]).to(torch.bfloat16)
    nan = [t for t in (0, T // 2) if t < T]
    bad = x.clone()
    bad[nan, 3] = float("nan")

    def run(x):
        ws = _poison((foe.workspace_bytes("cluster_block", foe.BF16, C, T, d, E, k, F),), torch.uint8)
        return foe.cluster_block(x, w["w_router"], None, w["w_gate"], w["w_up"], w["w_down"], k,
                                 ws=ws, out=torch.full((T, d), 7.0, dtype=torch.bfloat16,
                                                       device="cuda")).float().cpu()

    got, ref = run(bad), run(x)
    expect = ref.clone()
    expect[nan] = bad.float().cpu()[nan]  # C is a power of two: scale * C * x is x
    same = (got == expect) | (got.isnan() & expect.isnan())
    assert same.all(), (~same).nonzero()[:5]


@pytest.mark.parametrize("T,d,E,k,F,C,skew", [
    (128, 64, 8, 2, 64, 1, 0.0),      # 32 rows per expert: 8 parts
    (504, 72, 8, 1, 72, 1, 0.0),      # 63 rows, remainders of both widths
    (512, 72, 8, 1, 72, 1, 0.0),      # 64 rows: medium tiles
    (255, 264, 4, 1, 200, 3, 0.5),    # several clusters, skewed
    (2016, 72, 32, 1, 72, 1, 0.3),    # 4 and 8 parts, experts of 0 to over 256 rows
    (2016, 72, 32, 1, 72, 1, 9.0),    # all rows at one expert: 63 passes
    (260, 1032, 8, 1, 1000, 1, 0.0),  # 2 and 3 parts
    (40, 64, 1, 1, 64, 2, 0.0),       # one expert: 40 rows in two passes
])
def test_block_stream_parts(T, d, E, k, F, C, skew):
    """32 to 64 rows per expert: the weight stream with its passes of 32 rows dealt
    to parts of the grid."""
    print("block stream parts", T, d, E, k, F, C, skew, flush=True)
    bias = None if skew == 0 else (-skew * np.log(np.arange(1, E + 1))).astype(np.float32)
    inp = synth.make_block_inputs(dict(dtype="bf16", C=C, T=T, d=d, E=E, k=k, F=F, sigma=0.05,
                                       seed=3 * T + d, bias=None))
    for cl in inp["clusters"]:
        cl["bias"] = bias
    routes = bc.oracle_routes(inp["x"], inp["clusters"], k)
    assert not bc.exempt_mask(routes).any()
    ref, _, _ = bc.oracle_block(inp["x"], inp["clusters"], k, None, "renorm", routes=routes)
    w = {n: _dev(np.stack([cl[n] for cl in inp["clusters"]])).to(torch.bfloat16)
         for n in ("w_router", "w_gate", "w_up", "w_down")}
    ws = _poison((foe.workspace_bytes("cluster_block", foe.BF16, C, T, d, E, k, F),), torch.uint8)
    got = foe.cluster_block(_dev(inp["x"]).to(torch.bfloat16), w["w_router"],
                            None if bias is None else _dev(np.stack([bias] * C)), w["w_gate"],
                            w["w_up"], w["w_down"], k, ws=ws,
                            out=_poison((T, d), torch.bfloat16)).float().cpu().numpy()
    assert np.isfinite(got).all()
    e_out, e_upd = bc.block_errors(got, ref, inp["x"], C, None, "bf16")
    assert e_out <= bc.TOL["bf16"] and e_upd <= bc.TOL["bf16"], (e_out, e_upd)
