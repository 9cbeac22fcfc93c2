"""The host's rules for launch shapes (csrc/launch_plan.h), compiled by the host compiler and asked
without a GPU: on either side of each line the choice that was measured faster there."""
import ctypes as C
import shutil
import subprocess

import pytest

from paper_2510_10129_amd import build
from paper_2510_10129_amd._lib import LaunchOverride
from test_gpu_layer import CUT_SHAPES, FORCED_SHARES, SHARES_MODEL, UNEVEN_SHARES

CXX = shutil.which("g++") or shutil.which("c++")
pytestmark = pytest.mark.skipif(CXX is None, reason="no host C++ compiler")

SHIM = r"""
#include "launch_plan.h"
extern "C" {
void plan_attention(int n_cu, int n_row_tiles, int H_kv, int d_h, int t_max, int slots, int wide, int ovr, int* out) {
    const cc_attn_plan p = cc_plan_attention(n_cu, n_row_tiles, H_kv, d_h, t_max, slots, wide, ovr);
    out[0] = p.kind, out[1] = p.pieces, out[2] = p.ranges, out[3] = p.per_min;
}
int plan_gemm(int n_cu, int M, int N, int K, int64_t ws_floats, const cc_launch_override* ovr) {
    const cc_gemm_plan p = cc_plan_gemm(n_cu, M, N, K, K, K, ws_floats > 0, ws_floats, *ovr);
    return p.tile + 256 * p.shares;
}
int plan_gemm_duo(int n_cu, int M, int N, int K, int tile) {
    cc_launch_override o{};
    o.gemm_tile = tile;
    const cc_gemm_plan p = cc_plan_gemm(n_cu, M, N, K, K, K, false, 0, o);
    return p.duo ? p.tile : 0;
}
int plan_gemm_stream(int M, int N, int K, int64_t ws_floats) {
    const cc_gemm_plan p = cc_plan_gemm(256, M, N, K, K, K, ws_floats > 0, ws_floats, cc_launch_override{});
    return p.stream ? p.tile : 0;
}
int plan_gemm_staged_parts(int M, int N, int K, int64_t ws_floats) {
    const cc_gemm_plan p = cc_plan_gemm(256, M, N, K, K, K, ws_floats > 0, ws_floats, cc_launch_override{});
    return p.staged_parts ? p.tile : 0;
}
int norm_waves(int n_cu, int M, int d, int elem_bytes) { return cc_norm_waves(n_cu, M, d, elem_bytes); }
int asm_rows(int64_t n_rows, int width) { return cc_asm_rows(n_rows, width); }
int select_uses_ranges(int T) { return cc_select_uses_ranges(T); }
int plan_attn_workgroups(int n_cu, int64_t tiles, int64_t t_max) { return cc_plan_attn_workgroups(n_cu, tiles, t_max); }
}
"""
WHOLE, CUT, EVEN = 0, 1, 2


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "shim.cpp").write_text(SHIM)
    cmd = [CXX, "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", build.CSRC, "-I", build.ROOT + "/include",
           str(d / "shim.cpp"), "-o", str(d / "shim.so")]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
    return C.CDLL(str(d / "shim.so"))


def attn(plan, H_q, H_kv, d_h, N, M, n_cu=256, ovr=0, slots=None, wide=0):
    n_row_tiles, t_max = -(-M * (H_q // H_kv) // 256), -(-N // 64)
    plan.plan_attn_workgroups.argtypes = [C.c_int, C.c_int64, C.c_int64]
    slots = 2 * plan.plan_attn_workgroups(n_cu, n_row_tiles * H_kv, t_max) if slots is None else slots
    out = (C.c_int * 4)()
    plan.plan_attention(n_cu, n_row_tiles, H_kv, d_h, t_max, slots, wide, ovr, out)
    return tuple(out) + (slots,)


def gemm(plan, M, N, K, n_cu=256, ws_floats=32 << 20, **ovr):
    plan.plan_gemm.argtypes = [C.c_int, C.c_int, C.c_int, C.c_int, C.c_int64, C.POINTER(LaunchOverride)]
    if "gemm_tile" in ovr:
        ovr["gemm_tile"] = ord(ovr["gemm_tile"])
    r = plan.plan_gemm(n_cu, M, N, K, ws_floats, C.byref(LaunchOverride(**ovr)))
    return chr(r % 256), r // 256


def test_gemm_plans_fit_their_loops_and_workspace(plan):
    """Every plan over a wide range of sizes: loops that divide K, no share without a group of K ('t': a slice), shares of a
    round that fit one round and, in slots of their tiles, the workspace; a forced shape is taken wherever it has a loop for K."""
    for M in (1, 16, 64, 65, 200, 257, 883, 1523, 3404, 16576, 66000):
        for N in (64, 192, 512, 1536, 3584, 4096, 6144, 28672, 37888):
            for K in (64, 128, 192, 256, 448, 896, 1664, 1984, 3584, 4096, 8960, 14336, 18944):
                for ws in (0, 1 << 16, 4 << 20, 32 << 20):
                    tile, shares = gemm(plan, M, N, K, ws_floats=ws)
                    assert tile in ("bhst" if K % 128 == 0 else "bst") and 1 <= shares <= 16
                    bm, bn, slot = {"b": (256, 256, 65536), "h": (256, 128, 32768), "s": (128, 128, 0), "t": (64, 128, 8192)}[tile]
                    tiles = -(-M // bm) * -(-N // bn)
                    if shares > 1:
                        assert tile in "bht" and ws
                        last = tiles if tile == "t" else (tiles % 256 or 256)
                        assert last * shares <= 256 and last * shares * slot <= ws
                        assert K // (64 if tile == "t" else 128) >= shares and (tile == "t" or K % 128 == 0)
                for force in "bhst":
                    want = force if K % 128 == 0 or force in "bst" else None
                    assert gemm(plan, M, N, K, gemm_tile=force)[0] in ((want,) if want else ("b", "s"))


@pytest.mark.parametrize("M,N,K,tile", [
    (3000, 10880, 1984, "s"),           # three rounds of 256x256 tiles 179 us, four of 128x128 147
    (8320, 10880, 1984, "b"),           # 375, 394
])
def test_the_staged_loop_is_priced_by_its_own_rates(plan, M, N, K, tile):
    assert gemm(plan, M, N, K) == (tile, 1)


@pytest.mark.parametrize("M,N,K,tiles", [
    (5120, 2048, 256, "s"),             # short K, the ends of a tile count: 256x256 21.4 us, 128x128 18.4
    (8320, 2048, 256, "s"),             # 37.4, 24.9
    (6000, 1024, 1024, "bh"),           # one round of 128x128 tiles, two a CU: 35.1, one of 256x128 or 256x256 28
    (64, 28672, 4096, "t"),             # few rows: 45.7 us against 57.4
    (192, 28672, 4096, "h"),            # 98.7 thin, 74.9
    (64, 4096, 4096, "t"),              # 17.2, 22.3
    (192, 4096, 14336, "h"),            # 62 thin, 50.8 in shares of 256x256, 45.3 of 256x128
    (192, 6144, 4096, "h"),             # 33.0 thin, 35.2, 30.4
    (176, 10240, 8192, "h"),            # 59.7 thin, 58.0, 53.8
    (1280, 3584, 3584, "b"),            # 55.2 in shares of 256x256, 65.5 in 256x128
    (1152, 2880, 2880, "t"),            # 39.6, 54.5 in 128x128
    (2048, 1024, 4096, "t"),            # 31.4, 39.0 in shares of 256x128
    (3404, 28672, 4096, "b"),
    (16576, 28672, 4096, "b"),
])
def test_gemm_tile_is_the_one_measured_faster(plan, M, N, K, tiles):
    assert gemm(plan, M, N, K)[0] in tiles


@pytest.mark.parametrize("H_q,H_kv,d_h,N,M,kind", [
    (64, 8, 128, 330, 256, WHOLE),      # 20.5 us against 21.1 cut and 26.8 in even ranges
    (64, 8, 128, 592, 512, WHOLE),      # 26.4, 29.1, 33.6
    (64, 8, 128, 2112, 1024, WHOLE),    # 56.5, 63.6, 64.9
    (64, 8, 128, 6000, 1536, WHOLE),    # 158, 158, 168 (384 blocks)
    (4, 2, 64, 70, 16, WHOLE),          # 7.6, 9.2, 10.3
    (12, 12, 64, 170, 32, WHOLE),       # 8.8, 9.9 cut
    (64, 8, 128, 1104, 16, CUT),        # 29.6, 14.5, 15.6
    (64, 8, 128, 1104, 256, CUT),       # 35.5, 27.5, 28.8
    (32, 8, 128, 592, 64, CUT),         # 25.5, 15.9, 18.2
    (32, 8, 64, 850, 512, CUT),         # 24.1, 18.3, 24.3
    (32, 32, 128, 20000, 16, CUT),      # 363, 62, 67
    (4, 2, 64, 12000, 64, EVEN),        # 185, 33.8, 22.0
    (64, 8, 128, 4224, 512, EVEN),      # 92, 64, 57
    (28, 4, 128, 20000, 1536, EVEN),    # 390, 254, 213
])
def test_attention_grid_is_the_one_measured_faster(plan, H_q, H_kv, d_h, N, M, kind):
    assert attn(plan, H_q, H_kv, d_h, N, M)[0] == kind


@pytest.mark.parametrize("shape", CUT_SHAPES)
def test_shapes_of_the_cut_grid_tests_are_cut(plan, shape):
    assert attn(plan, *shape)[0] == CUT


@pytest.mark.parametrize("n_cu,kind", [(256, EVEN), (64, EVEN), (32, WHOLE)])
def test_attention_grid_follows_the_number_of_compute_units(plan, n_cu, kind):
    """64 blocks over 4096 slots: a quarter of 256 compute units, two rounds of 32."""
    got, _, ranges, _, slots = attn(plan, 32, 8, 128, 4096, 512, n_cu)
    assert got == kind and ranges in (0, n_cu) and slots == 2 * n_cu


def test_wide_token_strides_are_cut_but_not_into_even_ranges(plan):
    assert attn(plan, 8, 1, 128, 4096, 64)[0] == EVEN
    assert attn(plan, 8, 1, 128, 4096, 64, wide=1)[:2] == (CUT, 8)
    assert attn(plan, 8, 1, 128, 4096, 64, wide=1, ovr=3)[:2] == (CUT, 3)
    assert attn(plan, 8, 1, 128, 4096, 64, wide=1, ovr=1)[0] == WHOLE
    assert attn(plan, 8, 1, 128, 4096, 64, wide=1, ovr=64, slots=6)[:2] == (CUT, 3)


def test_attention_plans_fit_their_workspace(plan):
    """Every plan over a wide range of sizes: pieces and ranges within the slots and, for a cut grid, one
    round of workgroups, no empty runs by construction, and no piece shorter than the tiles allow."""
    for n_cu in (32, 256):
        for H_q, H_kv in ((1, 1), (4, 2), (28, 4), (64, 8), (32, 32), (96, 96)):
            for N in (1, 64, 65, 200, 1000, 4096, 33000, 131072, 1000000):
                for M in (1, 7, 64, 257, 1024, 5000, 20000):
                    for ovr, wide in ((0, 0), (1, 0), (2, 0), (64, 0), (0, 1), (1, 1), (3, 1), (64, 1)):
                        for slots in (None, 2, 6):              # more rows than the context was made for: fewer slots
                            kind, pieces, ranges, per_min, have = attn(plan, H_q, H_kv, 128, N, M, n_cu, ovr, slots, wide)
                            n_wg = -(-M * (H_q // H_kv) // 256) * H_kv
                            if kind == CUT:
                                assert 2 <= pieces <= -(-N // 64) and n_wg * pieces <= have
                                assert ovr or (pieces <= 8 and n_wg * pieces <= n_cu)
                            elif kind == EVEN:
                                assert 1 <= ranges <= have // 2 and per_min >= 1
                                assert ovr or ranges <= n_cu
                            assert kind == WHOLE or ovr != 1
                            assert not (wide and kind == EVEN)


@pytest.mark.parametrize("T,tiled", [(1, False), (16385, False), (20000, False), (24000, True), (131072, True)])
def test_selection_is_tiled_where_that_was_measured_faster(plan, T, tiled):
    assert bool(plan.select_uses_ranges(T)) == tiled


@pytest.mark.parametrize("M,d,elem_bytes,waves", [
    (16384, 576, 4, 1), (4096, 1024, 4, 1), (64, 1024, 2, 1),      # 13.2 us against 15.5; 7.9, 8.3
    (884, 4096, 2, 4), (64, 8192, 4, 4), (16384, 4096, 4, 4),      # 7.3, 9.8; 6.4, 11.2; 76, 84
    (4096, 4096, 2, 1), (8192, 2048, 2, 1), (16384, 1088, 2, 1),   # 15.3, 17.1; 15.0, 16.3; 18.7, 21.1
    (12000, 4096, 2, 4), (3000, 8192, 2, 2), (6000, 8192, 2, 4),   # 36.9, 39.0; 19.3, 22.0; 38.9, 39.5
    (16384, 16384, 2, 4),
])
def test_waves_of_a_row_norm(plan, M, d, elem_bytes, waves):
    assert plan.norm_waves(256, M, d, elem_bytes) == waves


def test_norm_plans_have_a_kernel(plan):
    """One wave holds rows of up to 4096 bf16 or 1024 fp32 elements, two up to 8192."""
    for d in range(64, 16385, 64):
        for M in (1, 64, 2048, 2049, 4096, 4097, 10240, 10241, 70000):
            assert plan.norm_waves(256, M, d, 2) in ((1, 2, 4) if d <= 4096 else (2, 4) if d <= 8192 else (4,))
            assert plan.norm_waves(256, M, d, 4) in ((1, 4) if d <= 1024 else (4,))


@pytest.mark.parametrize("n_rows,width,rows", [
    (1072, 1024, 4), (1072, 4096, 4), (4144, 1024, 8), (65584, 1024, 8),        # 7.2 us against 7.7 and 9.7; 94 against 99
    (28720, 4096, 8), (65584, 4096, 8), (16432, 512, 16), (65584, 64, 16),      # 186 and 420 against 200 and 459
])
def test_rows_of_an_assembly_wave(plan, n_rows, width, rows):
    plan.asm_rows.argtypes = [C.c_int64, C.c_int]
    assert plan.asm_rows(n_rows, width) == rows


@pytest.mark.parametrize("M,N,K,tile,duo", [
    (883, 4096, 4096, "s", True), (883, 6144, 4096, "h", True),        # 44.0 us against 59.8 in the ring loop, 63 against 79.9
    (1523, 4608, 3584, "h", True), (128, 4096, 14336, "s", True),      # 61, 80.8; 141, 168
    (3404, 2048, 256, "s", False),                                     # 19, 14.5 (two tiles a CU)
    (300, 512, 1984, "s", False),                                      # K % 128: the staged loop
])
def test_loop_of_the_smaller_tiles(plan, M, N, K, tile, duo):
    assert bool(plan.plan_gemm_duo(256, M, N, K, ord(tile))) == duo


@pytest.mark.parametrize("M,N,K,stream", [
    (64, 4096, 14336, True), (64, 28672, 4096, True), (64, 4096, 4096, True),      # six layers in a row 127.1 us each, 136.3 through the caches
    (8, 6144, 4096, True), (64, 16384, 2048, True), (64, 768, 3072, True),         # 107.6, 116.9; d = 2048 78.7, 81.0; 768 58.9, 60.7
    (64, 3456, 576, False), (64, 512, 2048, False), (8, 768, 512, False),          # 54.9, 53.8; 50.8, 48.5; 42.0, 39.9
    (65, 28672, 4096, False),                                                      # two row tiles
])
def test_weights_go_past_the_caches_where_that_was_measured_faster(plan, M, N, K, stream):
    plan.plan_gemm_stream.argtypes = [C.c_int, C.c_int, C.c_int, C.c_int64]
    assert bool(plan.plan_gemm_stream(M, N, K, 32 << 20)) == stream


@pytest.mark.parametrize("M,N,K,staged", [
    (65, 8192, 28672, True), (128, 8192, 28672, True),                   # 93.2 us against 123 from the accumulators; 104, 125
    (300, 3584, 18944, True), (448, 3584, 18944, True),                  # 68.3, 79.0; 76.2, 81.7
    (480, 4096, 14336, False), (512, 4096, 14336, False),                # 71.2, 67.6; 73.4, 70.5
    (3404, 28672, 4096, False),                                          # 4 % of the rows past M
    (64, 4096, 4096, False),                                             # thin tiles
])
def test_sums_of_shares_go_through_lds_where_that_was_measured_faster(plan, M, N, K, staged):
    plan.plan_gemm_staged_parts.argtypes = [C.c_int, C.c_int, C.c_int, C.c_int64]
    assert plan.plan_gemm_staged_parts(M, N, K, 32 << 20) == (ord("b") if staged else 0)


@pytest.mark.parametrize("shape,tile,n", list(zip(UNEVEN_SHARES, "thb", (3, 7, 8))))
def test_shapes_of_the_unequal_share_tests_are_cut(plan, shape, tile, n):
    M, d, f = shape
    assert gemm(plan, M, d, f, ws_floats=min(32 << 20, 8 * M * -(-2 * f // 256) * 256)) == (tile, n)


@pytest.mark.parametrize("M,N,K,tile,n", [
    (1523, 3584, 18944, "b", 3),        # 84 tiles, 148 groups: 2 equal shares 203 us, 173
    (448, 3584, 18944, "b", 9),         # 101.6, 80
    (3404, 6144, 4096, "b", 3),         # a full round and 80 tiles: 171.7, 166.4
    (883, 1536, 8960, "h", 5),          # 49.7, 41.3
    (64, 10240, 8192, "t", 3),          # 44.0, 38.6
])
def test_unequal_shares_where_they_were_measured_faster(plan, M, N, K, tile, n):
    assert gemm(plan, M, N, K) == (tile, n)


@pytest.mark.parametrize("tile,shares,M,M_cap", FORCED_SHARES)
def test_shapes_of_the_forced_share_tests_are_cut(plan, tile, shares, M, M_cap):
    """Every projection of those tests in as many shares as forced, but for grids that leave no room for them."""
    m, got = SHARES_MODEL, []
    ws = min(32 << 20, 8 * M_cap * -(-max(2 * m.f, m.n_qkv) // 256) * 256)
    for N, K in ((m.n_qkv, m.d), (m.d, m.H_q * m.d_h), (2 * m.f, m.d), (m.d, m.f)):
        assert K % 128 == 0
        got.append(gemm(plan, M, N, K, ws_floats=ws, gemm_tile=tile, gemm_splitk=shares))
    fit = M <= 300 or tile == "h"
    assert got[0] == got[2] == ((tile, shares) if fit else (tile, 1)) and (tile, shares) in got, got
    if M > 4000:                        # a full round ahead of the tiles in shares
        assert -(-M // 256) * -(-m.n_qkv // 128) > 256 and -(-M // 256) * -(-2 * m.f // 128) > 256
