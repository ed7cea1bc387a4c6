"""The rules that choose kernels and launch shapes by sizes (csrc/vnm_rules.h), compiled for the host and compared with
the measurements their comments state."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2410_16135_amd", "csrc")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    """rule("f(1, 2)") evaluates an expression on the rules and returns it as an integer."""
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not found")
    tmp = tmp_path_factory.mktemp("rules")

    def run(expr):
        src = tmp / "rule.cpp"
        src.write_text('#include "vnm_rules.h"\n#include <cstdio>\nusing namespace vnm;\n'
                       'int main() { std::printf("%%lld", (long long)(%s)); }\n' % expr)
        exe = str(tmp / "rule")
        res = subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", exe], capture_output=True, text=True)
        assert res.returncode == 0, res.stderr
        return int(subprocess.run([exe], capture_output=True, text=True, check=True).stdout)
    return run


# small matrices: a pass over the rows no wider than they need, a workgroup per row; tall ones: wide passes, 16 rows
@pytest.mark.parametrize("out,inn,aligned,waves,flight,rows", [
    (1, 64, 1, 4, 1, 1), (33, 64, 1, 4, 4, 1), (200, 304, 1, 4, 4, 1), (384, 11008, 1, 4, 4, 8), (500, 4096, 1, 4, 8, 4), (1000, 1000, 1, 4, 8, 1),
    (1024, 1024, 1, 4, 8, 1), (1025, 1025, 0, 16, 8, 4), (2048, 4096, 1, 8, 8, 8), (4096, 4096, 1, 16, 8, 16),
    (16, 1031, 0, 16, 8, 1), (11008, 64, 1, 16, 8, 8)])
def test_ria_score_shapes(rule, out, inn, aligned, waves, flight, rows):
    assert rule("colsum_shape(%d, %d).waves" % (out, aligned)) == waves
    assert rule("colsum_shape(%d, %d).flight" % (out, aligned)) == flight
    assert rule("score_rows(%d, %d)" % (out, inn)) == rows


# (T, out, column blocks, M) on both sides of the rule; the comments are the scalar and the other kernel's times in us
@pytest.mark.parametrize("T,out,B,M,scalar", [
    (1, 128, 1, 255, 1), (1, 4096, 4, 16, 1),           # 2.2 / 3.9, 3.6 / 3.7
    (1, 1000, 17, 64, 0), (1, 4096, 17, 255, 0),        # 9.3 / 3.2, 9.5 / 3.4
    (24, 128, 2, 64, 1), (31, 4096, 4, 16, 1),          # 2.9 / 7.0, 4.0 / 12.0
    (24, 1000, 33, 32, 0), (31, 4096, 32, 128, 0),      # 22.9 / 6.1, 25.0 / 13.6
    (32, 16, 17, 255, 1), (1024, 16, 17, 255, 1),       # 10.1 / 44.2, 11.0 / 45.5
    (333, 1000, 5, 255, 1), (64, 4096, 17, 255, 1),     # 6.6 / 16.6, 13.6 / 46.3
    (333, 1000, 148, 7, 0), (4096, 384, 24, 64, 0),     # 230 / 25.7, 162 / 47
    (1024, 4096, 17, 255, 0), (4096, 128, 19, 7, 0),    # 192 / 118, 27.6 / 6.9
    (40, 4096, 64, 64, 0), (333, 384, 24, 64, 0)])      # 63.7 / 37.1, 21.6 / 15.9
def test_scalar_kernel_where_there_are_few_column_blocks(rule, T, out, B, M, scalar):
    assert rule("plain_scalar_faster(%d, %d, %d, %d)" % (T, out, B, M)) == scalar


# rows per wave change at 512 workgroups, blocks per chunk at 64 blocks, 256 columns and one block
@pytest.mark.parametrize("T,out,M,blocks,rows", [
    (32, 1, 4, 64, 1), (128, 32 * 511, 7, 36, 1), (128, 32 * 511 + 1, 7, 36, 2), (128, 64 * 511, 128, 2, 2),
    (128, 64 * 511 + 1, 129, 1, 4), (11008, 4096, 255, 1, 4)])
def test_many_token_plan(rule, T, out, M, blocks, rows):
    assert rule("plain_plan(%d, %d, %d).blocks" % (T, out, M)) == blocks
    assert rule("plain_plan(%d, %d, %d).rows_per_wave" % (T, out, M)) == rows


MB = 1 << 20


# parts and weight within the L2s, the same XCD for writer and reader; the comments are the whole call with one result
# per thread and with four, in us
@pytest.mark.parametrize("T,out,pieces,weight,one_tile,wide", [
    (100, 8192, 5, 6.2, 1, 0), (256, 4096, 2, 6.0, 1, 0),       # 23.5 / 28.4, 16.5 / 18.5
    (128, 5120, 6, 4.6, 1, 0), (128, 16384, 3, 9.0, 1, 0),      # 24.0 / 25.7, 28.8 / 30.2
    (100, 8192, 6, 58.0, 1, 1), (128, 16384, 3, 57.0, 1, 1),    # 33.8 / 33.3, 36.4 / 34.2
    (100, 11008, 5, 17.0, 1, 1), (200, 8192, 3, 6.2, 0, 1),     # 28.8 / 27.8, 31.7 / 28.8
    (700, 4096, 2, 15.0, 0, 1), (24, 4096, 4, 15.0, 1, 0)])     # 43.4 / 40.7; below 2^19 results
def test_reduction_kernel(rule, T, out, pieces, weight, one_tile, wide):
    local = "parts_stay_in_l2(%d, %d, %d, %d, %d)" % (T, out, pieces, int(weight * MB), one_tile)
    assert rule("reduce_wide(%d, %d, %s)" % (T, out, local)) == wide


# token tiles, groups of 256 channels, K steps, pieces, MB of weight, MB of staged X, parts in their own L2
@pytest.mark.parametrize("tiles,groups,steps,pieces,weight,staged,in_l2,by_xcd", [
    (3, 16, 276, 5, 39, 10.1, 0, 1), (6, 16, 276, 2, 39, 20.2, 0, 1),          # 52.1 / 41.3, 73.1 / 67.6 us
    (9, 16, 276, 2, 39, 30.3, 0, 1), (7, 8, 172, 4, 12.1, 23.5, 0, 1),         # an odd number of tiles: 146 / 106, 67 / 44
    (16, 16, 276, 1, 39, 53.9, 0, 0), (32, 16, 103, 1, 14.5, 40.2, 0, 0),      # unsplit, every XCD has its tiles: 64.9 / 71.7
    (3, 16, 32, 5, 4.5, 1.9, 0, 0), (6, 32, 52, 1, 15, 4.0, 0, 0),             # 29.7 / 32.4, 39.0 / 40.2
    (11, 43, 64, 1, 25, 13.7, 0, 1), (3, 4, 128, 16, 4.5, 3.8, 0, 0),          # 61.2 / 52.9, 25.6 / 28.9
    (1, 32, 22, 5, 6.2, 0.7, 1, 0), (1, 16, 276, 13, 39, 3.4, 1, 0), (1, 16, 276, 13, 39, 3.4, 0, 0), (1, 43, 128, 5, 48, 1.3, 0, 1)])
def test_workgroup_order(rule, tiles, groups, steps, pieces, weight, staged, in_l2, by_xcd):
    assert rule("tiles_by_xcd(%d, %d, %d, %d, %d, %d, %d)" % (tiles, groups, steps, pieces, int(weight * MB), int(staged * MB), in_l2)) == by_xcd


# pieces, workgroups, steps of the last piece, row blocks, steps, M, column tables
@pytest.mark.parametrize("args,deep", [
    ((2, 192, 86, 64, 172, 8, 1), 1), ((2, 192, 32, 128, 64, 8, 1), 1), ((1, 132, 103, 172, 103, 5, 1), 0),
    ((2, 256, 52, 64, 103, 5, 1), 0), ((2, 192, 8, 24, 16, 8, 1), 1), ((2, 192, 7, 24, 15, 8, 1), 0),
    ((2, 192, 48, 64, 96, 7, 1), 1), ((2, 192, 47, 64, 95, 7, 1), 0),
    ((2, 192, 57, 64, 114, 9, 1), 1), ((2, 192, 52, 64, 103, 10, 1), 0), ((2, 192, 86, 64, 172, 8, 2), 0)])
def test_deep_loop(rule, args, deep):
    assert rule("deep_loop(%s)" % ", ".join(map(str, args))) == deep


# V, M, rows, columns; LDS of three workgroups per compute unit, and at least 160 workgroups (512 for eight steps)
@pytest.mark.parametrize("V,M,out,inn,steps", [
    (64, 8, 11008, 4096, 2), (32, 8, 11008, 4096, 4), (32, 9, 11008, 4096, 2), (128, 4, 11008, 4096, 2), (32, 4, 11008, 4096, 8),
    (64, 5, 4096, 4096, 2), (128, 10, 4096, 4096, 1), (32, 4, 1024, 1024, 4), (32, 8, 1024, 1024, 2), (32, 7, 1024, 1024, 4),
    (32, 4, 500, 4096, 4), (64, 5, 128, 160, 1)])
def test_scored_pruning_span(rule, V, M, out, inn, steps):
    blocks = -(-inn // M)
    assert rule("prune_scored_steps(%d, %d, %d, %d)" % (V, M, -(-out // V), -(-blocks // 8))) == steps


# 2^20 rows and more: rows are on grid.x for few tokens, 64 of them per workgroup on grid.y for many
@pytest.mark.parametrize("T,out,inn,fit", [
    (1, 1 << 20, 64, 1), (31, 1 << 26, 64, 1), (32, 1 << 20, 64, 1), (32, 64 * 65535, 64, 1), (32, 64 * 65535 + 1, 64, 0),
    (1, 64, 1 << 30, 0), (1, 64, (1 << 30) - 1, 1), (4096, 16, 64, 1)])
def test_sizes_of_the_plain_kernels(rule, T, out, inn, fit):
    assert rule("plain_sizes_fit(%d, %d, %d, 4)" % (T, out, inn)) == fit


# one to four tokens: the widest rows that whole tiles hold (16 waves up to 128 row blocks, then 8; up to 32 row blocks half
# tiles only), the widest that half tiles hold, three and four tokens up to 128 row blocks and 224 steps
@pytest.mark.parametrize("tokens,blocks,inn,steps,half,waves,takes", [
    (1, 65, 73664, 576, 0, 16, 1), (1, 65, 73672, 576, 0, 16, 0), (1, 129, 75200, 576, 0, 8, 1), (1, 129, 75208, 576, 0, 8, 0),
    (2, 100, 35264, 276, 0, 16, 1), (2, 100, 35272, 276, 0, 16, 0), (4, 128, 16064, 126, 0, 16, 1), (4, 128, 16072, 126, 0, 16, 0),
    (1, 64, 72640, 568, 1, 16, 1), (1, 64, 72648, 568, 0, 16, 1), (1, 33, 73664, 576, 0, 16, 1), (1, 32, 72648, 568, 1, 16, 0), (1, 32, 72640, 568, 1, 16, 1),
    (4, 64, 15040, 118, 1, 16, 1), (4, 64, 15048, 118, 0, 16, 1), (4, 20, 15048, 118, 1, 16, 0),
    (4, 129, 512, 8, 0, 8, 0), (4, 128, 8192, 224, 0, 16, 1), (4, 128, 8192, 225, 0, 16, 0), (2, 128, 8192, 225, 0, 16, 1),
    (1, 64, 4096, 80, 1, 8, 1), (1, 64, 4096, 81, 1, 16, 1), (1, 64, 4104, 65, 1, 16, 1)])
def test_one_to_four_tokens(rule, tokens, blocks, inn, steps, half, waves, takes):
    assert rule("gemv_half(%d, %d, %d)" % (tokens, blocks, inn)) == half
    assert rule("gemv_waves(%d, %d, %d, %d)" % (tokens, blocks, inn, steps)) == waves
    assert rule("gemv_takes(%d, %d, %d, %d)" % (tokens, blocks, inn, steps)) == takes


# on both sides of the line by results (T * out) and columns of X (steps * M), and the pieces above it
@pytest.mark.parametrize("T,out,pairs,steps,M,pieces", [
    (300, 1200, 15, 31, 4, 1), (300, 1200, 15, 32, 4, 17), (600, 1024, 20, 47, 5, 1), (600, 1024, 20, 48, 5, 12),
    (250, 8000, 64, 59, 5, 1), (250, 8000, 64, 60, 5, 3), (700, 3000, 72, 75, 5, 1), (700, 3000, 72, 76, 5, 3),
    (700, 4096, 96, 103, 5, 2), (500, 6000, 96, 83, 5, 1), (500, 6000, 96, 84, 5, 2), (1000, 3500, 112, 99, 5, 1), (1000, 3500, 112, 100, 5, 2),
    (1024, 4096, 128, 103, 5, 2), (2000, 2048, 128, 131, 5, 1), (2000, 2048, 128, 132, 5, 2),
    (504, 1205, 20, 14, 16, 12), (504, 1205, 20, 9, 12, 12), (800, 1407, 42, 18, 12, 1), (800, 1407, 42, 19, 12, 6), (842, 2000, 56, 26, 12, 1),
    (842, 2000, 56, 27, 12, 4), (1100, 448, 18, 15, 16, 14), (1100, 448, 18, 14, 16, 1), (900, 3000, 96, 41, 12, 1), (900, 3000, 96, 42, 12, 2),
    (1000, 4100, 136, 300, 5, 1), (1000, 4100, 136, 191, 12, 1), (1000, 4100, 136, 192, 12, 2), (100, 2048, 8, 10, 5, 25)])
def test_split_pieces(rule, T, out, pairs, steps, M, pieces):
    assert rule("split_pieces(%d, %d, %d, %d, %d)" % (T, out, pairs, steps, M)) == pieces


# K steps of a workgroup of the pruning inside a mask refresh (V, M, row blocks, steps)
@pytest.mark.parametrize("V,M,R,S,k", [(64, 5, 64, 103, 4), (32, 4, 128, 128, 8), (64, 8, 64, 64, 4), (64, 12, 64, 43, 2), (128, 16, 32, 32, 1),
                                       (128, 16, 2, 3, 1), (32, 5, 3, 3, 1), (64, 8, 16, 16, 1)])
def test_refresh_pruning_steps(rule, V, M, R, S, k):
    assert rule("prune_ria_steps(%d, %d, %d, %d)" % (V, M, R, S)) == k
    assert rule("prune_ria_lds(%d, %d, %d)" % (V, M, k)) <= 64 * 1024


def test_refresh_cases_reach_every_span(rule):
    from test_gpu_lora_merge import SPANS
    for out, inn, V, M, steps, batch in SPANS:
        R, S = -(-out // V), -(-(-(-inn // M)) // 8)
        assert rule("prune_ria_steps(%d, %d, %d, %d)" % (V, M, R, S)) == steps, (out, inn, V, M)
        assert rule("prune_batch(%d, %d)" % (V, min(256 // (steps * M), V))) == batch, (out, inn, V, M)
    assert {s[4] for s in SPANS} == {1, 2, 4, 8} and {s[5] for s in SPANS} == {4, 6, 8, 12}


# 8 steps at least, below 8 row blocks 56, or 24 at M = 8
@pytest.mark.parametrize("pieces,workgroups,blocks,steps,M,groups", [
    (1, 256, 64, 103, 5, 1), (1, 257, 64, 103, 5, 0), (2, 192, 64, 103, 5, 0), (1, 144, 64, 8, 5, 1), (1, 144, 8, 8, 5, 1), (1, 144, 64, 7, 5, 0),
    (1, 192, 64, 64, 10, 1), (1, 192, 64, 64, 11, 0), (1, 59, 4, 15, 5, 0), (1, 19, 4, 16, 7, 0), (1, 144, 7, 55, 5, 0), (1, 144, 7, 56, 5, 1),
    (1, 21, 1, 23, 8, 0), (1, 21, 1, 24, 8, 1)])
def test_two_wave_groups(rule, pieces, workgroups, blocks, steps, M, groups):
    assert rule("kgroups(%d, %d, %d, %d, %d)" % (pieces, workgroups, blocks, steps, M)) == groups


# (tiles, groups, steps, pieces, MiB of weight and staged X, one generation, 8 row blocks per workgroup, parts in L2) -> kind
# (0 grid order, 1 runs, 2 boxes) and parts of the token tiles
@pytest.mark.parametrize("args,kind,log_t", [
    ((16, 16, 103, 1, 17.6, 21.4, 1, 0, 0), 2, 2), ((3, 43, 103, 1, 47.0, 4.0, 1, 0, 0), 2, 0), ((1, 6, 103, 1, 6.0, 1.3, 1, 0, 0), 0, 0),
    ((99, 6, 12, 1, 2.7, 23.0, 0, 1, 0), 2, 3), ((99, 6, 12, 1, 2.7, 23.0, 0, 0, 0), 0, 0), ((32, 8, 103, 1, 17.6, 43.0, 0, 1, 0), 0, 0),
    ((9, 11, 276, 1, 47.0, 32.0, 0, 1, 0), 1, 0), ((6, 16, 103, 2, 17.6, 8.0, 0, 0, 0), 1, 0), ((1, 16, 103, 8, 17.6, 1.3, 0, 0, 1), 0, 0)])
def test_xcd_order(rule, args, kind, log_t):
    tiles, groups, steps, pieces, weight, staged, one, wide, in_l2 = args
    call = "xcd_order(%d, %d, %d, %d, %d, %d, %d, %d, %d)" % (tiles, groups, steps, pieces, int(weight * MB), int(staged * MB), one, wide, in_l2)
    assert rule(call + ".kind") == kind
    if kind == 2:
        assert rule(call + ".log_t") == log_t


# boxes in an unsplit launch of more than one generation: only with no generation more than an even share of the launch takes
# (the comments are runs or grid order / boxes, us), and where they save more the less even they are
@pytest.mark.parametrize("args,kind", [
    ((19, 12, 48, 1, 9.7, 17.8, 0, 1, 0), 1), ((18, 8, 20, 1, 2.5, 4.6, 0, 1, 0), 0),         # 43.8 / 61.1, 40.1 / 46.4
    ((44, 22, 22, 1, 8.3, 12.3, 0, 1, 0), 0), ((47, 5, 24, 1, 2.0, 23.0, 0, 1, 0), 2)])       # 200 / 210; 26.0 / 20.3
def test_boxes_only_where_they_are_even(rule, args, kind):
    tiles, groups, steps, pieces, weight, staged, one, wide, in_l2 = args
    assert rule("xcd_order(%d, %d, %d, %d, %d, %d, %d, %d, %d).kind" % (tiles, groups, steps, pieces, int(weight * MB), int(staged * MB), one, wide, in_l2)) == kind


# two wave groups where every grid of boxes gives an XCD more than 32 workgroups: columns, unless grid order fetches less
# (the comments are grid order / columns, us)
@pytest.mark.parametrize("tiles,groups,steps,weight,staged,kind", [
    (82, 3, 47, 1.1, 75.0, 3), (33, 7, 47, 4.1, 24.2, 3),           # 45.8 / 27.6, 36.0 / 24.9
    (49, 5, 59, 2.2, 56.5, 3), (12, 21, 24, 4.5, 4.5, 0), (16, 16, 103, 17.6, 21.4, 2)])
def test_columns_where_no_box_fits(rule, tiles, groups, steps, weight, staged, kind):
    assert rule("xcd_order(%d, %d, %d, 1, %d, %d, 1, 0, 0).kind" % (tiles, groups, steps, int(weight * MB), int(staged * MB))) == kind


# the columns cover every (token tile, group) once, an XCD at most one workgroup more than another
@pytest.mark.parametrize("tiles,groups", [(82, 3), (49, 5), (13, 17), (8, 31), (3, 85)])
def test_columns_cover_the_launch(tiles, groups):
    total = tiles * groups
    each, rest = total >> 3, total & 7
    ids = [(n & 7) * each + min(n & 7, rest) + (n >> 3) for n in range(total)]
    assert sorted((i // groups, i % groups) for i in ids) == [(t, g) for t in range(tiles) for g in range(groups)]


# the boxes cover every (token tile, group) once, and no XCD's box is larger than the launch provides for
@pytest.mark.parametrize("tiles,groups,log_t", [(9, 16, 0), (9, 16, 1), (12, 13, 2), (17, 1, 3), (99, 6, 3), (8, 8, 3), (5, 4, 1)])
def test_boxes_cover_the_launch(rule, tiles, groups, log_t):
    most, seen = rule("xcd_box_most(%d, %d, %d)" % (tiles, groups, log_t)), []
    for n in range(8 * most):
        xcd, lg = n & 7, 3 - log_t
        ct, cg = xcd & ((1 << log_t) - 1), xcd >> log_t
        t_lo, g_lo = (ct * tiles) >> log_t, (cg * groups) >> lg
        t_n, g_n = (((ct + 1) * tiles) >> log_t) - t_lo, (((cg + 1) * groups) >> lg) - g_lo
        row = (n >> 3) // t_n
        if row < g_n:
            seen.append((t_lo + (n >> 3) - row * t_n, g_lo + row))
    assert sorted(seen) == [(t, g) for t in range(tiles) for g in range(groups)]


# rows per thread up to 4, 6, 8 and 12, and two and three trips
@pytest.mark.parametrize("V,groups,batch", [(32, 8, 4), (64, 12, 6), (64, 8, 8), (64, 6, 12), (128, 16, 8), (64, 4, 8), (128, 6, 12), (128, 4, 12),
                                            (32, 32, 4), (128, 1, 12)])
def test_prune_batch(rule, V, groups, batch):
    assert rule("prune_batch(%d, %d)" % (V, groups)) == batch


# half tiles of one to four tokens: every quarter of a row block once, the four of a block on one XCD (workgroup n mod 8)
# except in the row blocks beyond a multiple of 8
@pytest.mark.parametrize("blocks", [1, 7, 8, 9, 16, 29, 64])
def test_half_tiles_cover_the_launch(blocks):
    grid, seen = 4 * blocks, {}
    for n in range(grid):
        by_xcd = n < (grid & ~31)
        rp, part = ((n >> 5) * 8 + (n & 7), (n >> 3) & 3) if by_xcd else (n >> 2, n & 3)
        seen.setdefault(rp, {})[part] = n & 7
    assert sorted(seen) == list(range(blocks)) and all(sorted(p) == [0, 1, 2, 3] for p in seen.values())
    assert all(len(set(p.values())) == 1 for rp, p in seen.items() if rp < blocks // 8 * 8)
