"""The rules that choose kernels by the lattice's size (host only, nothing is launched).

tests/dispatch_rules.cpp is built against the library and gives its rules C names.
"""
import ctypes
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

FP32, FP16 = 0, 1


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    from paper_1607_08675_amd import _capi, build
    if not os.path.exists(_capi.LIB_PATH):
        build.build()
    if not shutil.which("g++") or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("g++ or the HIP headers missing")
    out = str(tmp_path_factory.mktemp("rules") / "rules.so")
    pkg = os.path.dirname(_capi.LIB_PATH)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-I", "/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(pkg, "csrc"),
                    os.path.join(ROOT, "tests", "dispatch_rules.cpp"), _capi.LIB_PATH,
                    "-Wl,-rpath," + pkg, "-o", out], check=True)
    return ctypes.CDLL(out)


@pytest.mark.parametrize("nx,ny,esize,bypass", [
    (1024, 1024, 4, 0), (1448, 1448, 4, 1), (512, 512, 2, 1), (1021, 767, 4, 0),
    # narrow rows: few sites, many lines
    (16, 100000, 2, 1), (2, 100000, 4, 1), (33, 70000, 2, 1), (72, 40000, 2, 1)])
def test_stores_by_the_lines_that_the_rows_take(rules, nx, ny, esize, bypass):
    assert rules.rule_stores_bypass(nx, ny, esize, 0) == bypass


@pytest.mark.parametrize("nx,ny,esize,bypass", [
    (1024, 1024, 4, 1), (1000, 1000, 4, 1), (1500, 1500, 2, 1), (1100, 1100, 2, 1),
    (640, 640, 4, 0), (1024, 1024, 2, 0), (512, 512, 4, 0), (100, 100, 4, 1)])
def test_kept_states_go_past_the_cache_that_they_outgrow(rules, nx, ny, esize, bypass):
    assert rules.rule_stores_bypass(nx, ny, esize, 1) == bypass


@pytest.mark.parametrize("tiles,ny,rows", [
    (274, 33, 9), (274, 100, 25), (341, 40, 10), (274, 24, 8), (274, 2, 8),   # four strips
    (274, 250, 32),                               # taller than 128 rows: many rounds
    (342, 40, 40), (391, 33, 33), (469, 100, 100),   # one strip nearly fills a round
    (256, 40, 20), (196, 100, 50), (169, 40, 14), (16, 4096, 128), (8, 2048, 32)])
def test_one_strip_does_not_leave_half_the_card(rules, tiles, ny, rows):
    assert rules.rule_strip_rows(tiles, ny, 512, 8, 128, 32) == rows


@pytest.mark.parametrize("storage,most", [(FP32, 512), (FP16, 1024)])
@pytest.mark.parametrize("nx,ny", [(2, 2), (64, 64), (256, 256), (600, 600), (1024, 1024),
                                   (2500, 2500), (3000, 1999), (100000, 8), (120000, 33),
                                   (20000, 16), (200, 16000), (5000, 2900), (8192, 8192)])
def test_diagnostics_strips_fill_whole_rounds(rules, nx, ny, storage, most):
    tiles, rows = -(-nx // 256), rules.rule_diag(nx, ny, storage, 0)
    blocks = rules.rule_diag(nx, ny, storage, 1)
    assert 1 <= rows <= 64 and blocks == tiles * -(-ny // rows)
    assert blocks <= most or rows == 64
    assert not rules.rule_diag_by_row(nx, ny) or rows == 1


@pytest.mark.parametrize("nx,ny,storage,wide", [
    (4096, 4096, FP32, 1), (1448, 1448, FP32, 1), (8192, 8192, FP16, 1), (1000, 1000, FP32, 0),
    (56, 40000, FP32, 1), (112, 20000, FP32, 1), (168, 50000, FP16, 1), (100, 40000, FP32, 1),
    # one column of 56 and a few columns more
    (60, 40000, FP32, 0), (72, 40000, FP32, 0), (120, 50000, FP32, 0), (60, 100000, FP16, 0),
    (72, 100000, FP16, 0)])
def test_wide_tiles_where_they_issue_fewer_lanes(rules, nx, ny, storage, wide):
    assert rules.rule_tile_wide(nx, ny, storage, 5, 0) == wide
    assert rules.rule_tile_wide(nx, ny, storage, 3, 0) == 0


def test_wide_tiles_of_kept_states(rules):
    assert [rules.rule_tile_wide(nx, ny, FP32, 4, 1)
            for nx, ny in ((1024, 1024), (58, 20000), (64, 20000), (700, 700))] == [1, 1, 0, 0]
    assert not rules.rule_tile_wide(4096, 4096, FP16, 4, 1)


# low, wide lattices that leave most of the tiles' rows empty go by rows again
LOW = [(100000, 2), (1000000, 4), (400000, 12), (75000, 4), (50000, 6), (107142, 28)]


@pytest.mark.parametrize("storage", [FP32, FP16])
@pytest.mark.parametrize("nx,ny", LOW)
def test_low_lattices_go_by_rows(rules, nx, ny, storage):
    for les in (0, 1, 2, 3, 4, 6):
        assert rules.rule_tile_steps(nx, ny, storage, les) == 0
    for nb in (0, 1):
        assert not rules.rule_tile_keep(nx, ny, storage, nb)


@pytest.mark.parametrize("nx,ny,local,nb32,nb16", [
    (2, 2, 5, 3, 3), (64, 64, 5, 3, 3), (4096, 8, 5, 3, 3), (256, 256, 9, 3, 3),
    (1000, 100, 5, 3, 3), (6000, 50, 5, 3, 3), (1021, 767, 5, 3, 2), (1024, 1024, 5, 3, 2),
    (2, 100000, 5, 3, 3), (60, 40000, 5, 3, 2), (4096, 4096, 5, 0, 2), (8192, 8192, 5, 0, 2),
    (41666, 24, 5, 0, 2), (30000, 100, 5, 0, 2)])
def test_other_lattices_keep_their_tiles(rules, nx, ny, local, nb32, nb16):
    for les in (0, 1):
        assert rules.rule_tile_steps(nx, ny, FP32, les) == local
        assert rules.rule_tile_steps(nx, ny, FP16, les) == local
    for les in (2, 3, 4, 6):
        assert rules.rule_tile_steps(nx, ny, FP32, les) == nb32
    assert rules.rule_tile_steps(nx, ny, FP16, 6) == nb16


@pytest.mark.parametrize("n,les,k", [
    (3000, 4, 2), (3500, 4, 0), (8192, 4, 0), (4096, 2, 2), (6000, 3, 2), (8192, 2, 0),
    (8192, 3, 0), (8192, 6, 2), (8192, 1, 5)])
def test_fp16_closures_leave_the_tiles_on_large_lattices(rules, n, les, k):
    assert rules.rule_tile_steps(n, n, FP16, les) == k


@pytest.mark.parametrize("nx,ny,storage,nb,k,tiles", [
    (1000, 1000, FP32, 0, 2, 1), (1024, 1024, FP32, 0, 3, 0), (1448, 1448, FP16, 0, 2, 1),
    (1448, 1448, FP32, 1, 1, 1), (2048, 2048, FP32, 1, 1, 0), (64, 64, FP32, 0, 2, 1),
    # tiles whose second row of tiles is nearly empty
    (31250, 32, FP32, 0, 2, 0), (31250, 32, FP16, 0, 2, 0), (93750, 32, FP16, 0, 3, 0),
    (43100, 40, FP16, 1, 1, 0), (35714, 28, FP32, 1, 1, 0)])
def test_short_launches(rules, nx, ny, storage, nb, k, tiles):
    assert rules.rule_tile_short(nx, ny, storage, nb, k) == tiles


@pytest.mark.parametrize("nx,ny,storage,nb,keeps", [
    (1024, 1024, FP32, 0, 1), (1200, 1200, FP32, 0, 1), (2048, 2048, FP16, 0, 1),
    (512, 512, FP32, 1, 1), (1024, 1024, FP32, 1, 0), (1448, 1448, FP16, 1, 1),
    (64, 64, FP32, 1, 1), (53570, 56, FP16, 0, 0), (43100, 40, FP16, 1, 0), (100000, 8, FP16, 1, 0)])
def test_kept_states_by_size(rules, nx, ny, storage, nb, keeps):
    assert rules.rule_tile_keep(nx, ny, storage, nb) == keeps


@pytest.mark.parametrize("nx,ny,fp32,fp16", [
    (64, 64, 1, 1), (1024, 1024, 1, 1), (6000, 50, 1, 1), (1448, 1448, 1, 1), (1800, 1800, 1, 1),
    (10000, 300, 1, 1), (400, 8000, 1, 1), (60, 40000, 1, 1), (2048, 2048, 0, 1),
    (4096, 4096, 0, 0), (20000, 16, 0, 0),   # the last: more tiles than slots
    # the rows fill their rounds
    (8000, 400, 0, 1), (16000, 200, 0, 1), (2000, 1500, 0, 1), (4096, 512, 0, 1),
    (107142, 28, 0, 0)])
def test_reverse_tiles_where_rows_fill_their_rounds_badly(rules, nx, ny, fp32, fp16):
    assert rules.rule_adj_tile(nx, ny, FP32) == fp32
    assert rules.rule_adj_tile(nx, ny, FP16) == fp16


@pytest.mark.parametrize("nx,ny,nz", [(2, 2, 2), (96, 96, 96), (130, 130, 130), (160, 160, 160),
                                      (192, 192, 192), (200, 200, 200), (256, 256, 256),
                                      (64, 4, 4000), (3072, 64, 7), (4000, 300, 5)])
def test_3d_diagnostics_take_one_round(rules, nx, ny, nz):
    tiles = -(-nx // 64) * -(-ny // 4)
    chunk = rules.rule_diag3_chunk(tiles, nz)
    assert 1 <= chunk <= nz
    blocks = tiles * -(-nz // chunk)
    assert blocks <= 768 or (tiles > 768 and chunk == nz)
    assert chunk == 1 or tiles * -(-nz // (chunk - 1)) > 768 or blocks == tiles   # no fewer planes would do
