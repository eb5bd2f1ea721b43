"""Renormalised routing of several clusters against the oracle on both sides of
the rule between one pass over x and a workgroup per cluster, past 64 score
columns and with many tokens; and the dispatch that takes its expert counts."""

import numpy as np
import pytest

import oracle
from paper_2605_06206_amd import foe, synth
from test_gpu_parity import TOL, _block_gpu, _check_block, check_route, host, say, to_dev

pytestmark = pytest.mark.gpu


SIZES = [(C, E, T, d) for C, E in ((8, 32), (5, 14), (20, 4), (2, 128), (64, 4))
         for T, d in ((2048, 136), (4100, 72), (9000, 264))]


# (x of 4104 columns: per cluster and in one pass)
@pytest.mark.parametrize("C,E,T,d", SIZES + [(5, 14, 2100, 4104), (20, 4, 2100, 4104)])
@pytest.mark.parametrize("dt,bias", [("bf16", True), ("bf16", False), ("f32", True)])
def test_route_clusters_past_64_columns(C, E, T, d, dt, bias):
    say("route clusters", C, E, T, d, dt, bias)
    k = min(3, E)
    rng = np.random.default_rng([C, T, E])
    xs = rng.standard_normal((T, d)).astype(np.float32)
    wr = (rng.standard_normal((C, E, d)) / np.sqrt(d)).astype(np.float32)
    if dt == "bf16":
        xs, wr = synth.round_to_bf16(xs), synth.round_to_bf16(wr)
    bs = (rng.standard_normal((C, E)) * 0.1).astype(np.float32) if bias else None
    gidx, gw = foe.route(to_dev(xs, dt), to_dev(wr, dt), to_dev(bs, "f32") if bias else None, k)
    gidx, gw = host(gidx).reshape(C, T, k), host(gw).reshape(C, T, k)
    for h in range(0, C, 1 if C <= 8 else 7):
        ref = oracle.route(xs, wr[h], bs[h] if bias else None, k)
        check_route(gidx[h], gw[h], ref, TOL[dt])


@pytest.mark.parametrize("T,d,E,k,F,C,bias", [
    (4100, 64, 14, 2, 64, 5, "zipf1.2"),   # per cluster; counts of 16-token blocks
    (8200, 64, 40, 1, 64, 2, None),        # per cluster, streaming blocks of 32 tokens
    (4100, 4096, 4, 2, 8, 20, None),       # one pass
    (2048, 64, 32, 2, 64, 4, None),        # 4096 pairs a cluster: one index workgroup
    (4096, 64, 8, 1, 64, 2, "zipf1.2"),
    (4097, 64, 8, 1, 64, 2, None),         # 4097: the routing kernel's counts
])
def test_block_takes_the_counts_of_either_side(T, d, E, k, F, C, bias):
    say("block counts", T, d, E, k, F, C, bias)
    cfg = dict(dtype="bf16", C=C, T=T, d=d, E=E, k=k, F=F, sigma=0.05, seed=T + E, bias=bias)
    inp = synth.make_block_inputs(cfg)
    _check_block(inp, _block_gpu(inp))
