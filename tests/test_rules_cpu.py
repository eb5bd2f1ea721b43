"""The rules that pick a kernel by sizes alone (csrc/rules.hpp), compiled for the
host."""

import ctypes
import shutil
import subprocess

import pytest

from paper_2605_06206_amd import build as build_mod


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not found")
    tmp = tmp_path_factory.mktemp("rules")
    (tmp / "r.cpp").write_text(
        '#include "rules.hpp"\n'
        'extern "C" int per_cluster(int bf16, int C, int T, int d, int E) {\n'
        '  return foe::route_per_cluster(bf16 != 0, C, T, d, E);\n}\n'
        'extern "C" int form(int E, int d, int F, long long rows) {\n'
        '  return (int)foe::ffn_form(E, d, F, rows, 256);\n}\n'
        'extern "C" int f32_tiled(int d, int F, long long gather_rows) {\n'
        '  return foe::f32_tiled(d, F, gather_rows);\n}\n'
        'extern "C" int spreads(int C, int E, int R, int d, int F) {\n'
        '  return foe::stream_spreads(C, E, R, d, F, 256);\n}\n'
        'extern "C" int parts(int R, int E, int wgs) {\n'
        '  return foe::stream_parts(R, E, wgs, 256);\n}\n')
    lib = str(tmp / "r.so")
    subprocess.run([gxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", build_mod.CSRC,
                    str(tmp / "r.cpp"), "-o", lib], check=True)
    return ctypes.CDLL(lib)


# (dtype, C, E, T, d, us in one pass, us with a workgroup per cluster), measured
ROUTE = [
    ("bf16", 8, 8, 1, 2048, 15.9, 6.3),
    ("bf16", 8, 8, 1000, 2048, 15.3, 9.8),
    ("bf16", 8, 8, 2040, 7168, 37.1, 43.1),
    ("bf16", 8, 4, 2040, 4096, 16.2, 23.8),
    ("bf16", 16, 2, 1000, 7168, 26.3, 36.4),
    ("bf16", 2, 40, 32768, 2048, 155.5, 63.2),
    ("bf16", 20, 4, 32768, 2048, 291.6, 413.5),
    ("bf16", 20, 4, 4096, 4096, 48.1, 104.1),
    ("bf16", 8, 10, 4096, 4096, 35.7, 50.8),
    ("bf16", 8, 16, 2048, 2048, 28.9, 17.8),
    ("bf16", 8, 16, 4096, 4096, 44.7, 59.1),
    ("bf16", 4, 32, 32768, 4096, 334.3, 190.9),
    ("bf16", 8, 32, 8192, 2048, 95.9, 41.9),
    ("bf16", 8, 32, 32768, 4096, 635.3, 368.8),
    ("bf16", 64, 2, 256, 4096, 104.7, 22.3),
    ("bf16", 64, 2, 8192, 4096, 204.9, 632.7),
    ("bf16", 64, 4, 32768, 4096, 1346.6, 2561.5),
    ("f32", 8, 4, 2040, 2048, 19.4, 27.7),
    ("f32", 16, 2, 1000, 2048, 21.6, 27.4),
    ("f32", 8, 16, 2048, 2048, 80.5, 33.3),
    ("f32", 4, 32, 32768, 2048, 298.8, 373.1),
    ("f32", 64, 2, 32768, 2048, 475.7, 2479.9),
    ("f32", 2, 128, 32768, 2048, 840.3, 567.9),
]


@pytest.mark.parametrize("dt,C,E,T,d,one,per", ROUTE)
def test_routing_of_several_clusters_takes_the_faster_side(rules, dt, C, E, T, d, one, per):
    assert bool(rules.per_cluster(int(dt == "bf16"), C, T, d, E)) == (per < one)


def test_routing_rule_at_its_ends(rules):
    for bf16 in (0, 1):
        for T in (1, 2047, 2048, 1 << 30):
            assert not rules.per_cluster(bf16, 1, T, 2048, 16)      # one cluster
        for T in (2048, 4096, 8192, 65536):
            assert not rules.per_cluster(bf16, 8, T, 2048, 8)       # 64 columns, many tokens
        assert rules.per_cluster(bf16, 64, 1, 8, 4)
        assert rules.per_cluster(bf16, 64, 1, 1 << 20, 4)


# (C, E, pairs per cluster, d, F, us with medium tiles, us with the stream in
# parts), uniform router, measured on 256 CUs
STREAM = [
    (1, 8, 320, 384, 384, 32.8, 22.9),
    (2, 8, 384, 1024, 384, 40.6, 27.5),
    (1, 12, 576, 1280, 512, 44.7, 32.3),
    (2, 16, 768, 384, 256, 36.3, 26.4),
    (1, 16, 1008, 1024, 640, 42.7, 48.2),
    (4, 8, 504, 384, 1024, 44.8, 49.8),
    (1, 24, 1344, 640, 640, 42.2, 46.0),
]


@pytest.mark.parametrize("C,E,R,d,F,mid,stream", STREAM)
def test_32_to_64_rows_take_the_faster_form(rules, C, E, R, d, F, mid, stream):
    assert bool(rules.spreads(C, E, R, d, F)) == (stream < mid)


def test_stream_parts_at_their_ends(rules):
    assert not rules.spreads(1, 8, 255, 64, 64) and rules.spreads(1, 8, 256, 64, 64)
    assert rules.spreads(1, 8, 511, 64, 64) and not rules.spreads(1, 8, 512, 64, 64)
    assert rules.spreads(1, 32, 1024, 64, 128) and not rules.spreads(1, 32, 1024, 64, 129)
    assert rules.parts(255, 8, 8) == 1          # under 32 rows per expert
    assert rules.parts(256, 8, 8) == 8
    assert rules.parts(256, 8, 37) == 6
    assert rules.parts(256, 8, 128) == 2
    assert rules.parts(256, 8, 4096) == 1


STREAMED, MID, LARGE, FUSED = range(4)
# (experts, rows, d, F, us with medium tiles, with large ones, with large ones in one
# launch), measured on 256 CUs; the last two rows with a skewed router
FORMS = [
    (24, 1728, 1024, 1024, 57.0, 62.2, 82.9),
    (40, 2880, 1536, 1024, 122.7, 134.0, 144.0),
    (64, 6080, 4096, 256, 213.3, 235.2, 226.4),
    (16, 1776, 2048, 512, 57.8, 75.6, 75.2),
    (4, 2288, 1024, 384, 44.5, 67.5, 62.4),
    (12, 5400, 2048, 384, 77.1, 93.4, 99.1),
    (16, 4096, 2048, 1024, 127.0, 119.0, 138.0),
    (16, 5120, 4096, 256, 111.0, 145.0, 139.0),
    (32, 5832, 2048, 704, 131.0, 113.6, 127.6),
    (32, 2048, 2048, 2048, 200.4, 240.0, 233.7),
    (24, 3072, 2048, 1024, 148.2, 119.3, 127.0),
    (12, 3684, 768, 1536, 72.0, 114.0, 102.0),
    (64, 10240, 5120, 512, 526.2, 376.9, 360.8),
    (40, 6400, 2048, 1024, 236.5, 233.8, 218.1),
    (48, 12096, 2560, 640, 267.7, 253.0, 209.3),
    (8, 15168, 4096, 256, 230.1, 218.5, 198.9),
    (64, 28800, 2048, 384, 328.9, 302.4, 252.7),
    (64, 27584, 4096, 1024, 1412.9, 1040.0, 860.5),
    (48, 21600, 4096, 256, 414.8, 341.9, 294.5),
    (64, 4096, 2560, 1536, 410.2, 360.3, 346.5),
]


@pytest.mark.parametrize("E,rows,d,F,mid,large,fused", FORMS)
def test_expert_ffn_takes_the_fastest_form(rules, E, rows, d, F, mid, large, fused):
    us = {MID: mid, LARGE: large, FUSED: fused}
    assert rules.form(E, d, F, ctypes.c_longlong(rows)) == min(us, key=us.get)


def test_expert_ffn_forms_at_their_ends(rules):
    def form(E, rows, d, F):
        return rules.form(E, d, F, ctypes.c_longlong(rows))

    assert form(16, 511, 2048, 1024) == STREAMED and form(16, 512, 2048, 1024) == MID
    assert form(2, 191, 64, 65536) == MID      # under 96 rows: whatever the tiles
    assert form(2, 192, 64, 65536) == FUSED
    assert form(2, 1 << 30, 8, 8) == FUSED     # many tiles, little work
    assert form(64, 6143, 1 << 14, 1 << 12) == FUSED
    assert form(1, 1 << 31, 8, 8) == FUSED     # rows past 32 bits


def test_fp32_operands_past_32_bit_offsets_take_the_plain_kernels(rules):
    def tiled(d, F, rows):
        return bool(rules.f32_tiled(d, F, ctypes.c_longlong(rows)))

    assert tiled(8, 8, 0) and tiled(1024, 512, 1 << 18)
    # 64 rows of an operand, every one of them below 2 GiB
    assert tiled(8388600, 8, 0) and not tiled(8388608, 8, 0)
    assert tiled(8, 8388600, 0) and not tiled(8, 8388608, 0)
    # the whole gathered source
    assert tiled(1024, 512, (1 << 19) - 1) and not tiled(1024, 512, 1 << 19)
    assert tiled(1024, 512, 0)
    assert not tiled(8, 8, 1 << 31)
