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
