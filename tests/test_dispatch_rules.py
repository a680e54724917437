"""The rules that choose kernels and cut work, evaluated on the host (tests/dispatch_rules.py)."""
import os
import random

import pytest

from paper_2511_19797_amd import binding, build as tvm_build
from tests import dispatch_cases as dc
from tests.dispatch_rules import ask

MAX_ROWS = 2 ** 31 - 1   # the largest row count a descriptor may name


@pytest.mark.parametrize("rows", [64, 1024, 1089, 2 ** 29 - 1, 2 ** 29, 2 ** 30 + 17, 2 ** 31 - 64, 2 ** 31 - 63, MAX_ROWS])
def test_parts_cover_the_rows_in_order(rows):
    """Every part starts where the one before ends, in whole tiles of 64, at the tile floor(z * tiles / parts) in exact
    arithmetic, up to the largest row count."""
    tiles = -(-rows // 64)
    for parts in (2, 3, 7, 127, 128, 255, 256):
        if parts > tiles:
            continue
        got = ask([("part_rows", rows, z, parts) for z in range(parts)])
        assert got == [(z * tiles // parts * 64, min(rows, (z + 1) * tiles // parts * 64)) for z in range(parts)]


def test_rules_at_the_largest_row_counts():
    """One (batch, head) with up to 2^31 - 1 rows on a side: no overflow on the way to the answer."""
    assert ask([("bwd_splits", 1, MAX_ROWS, 4096, 4), ("bwd_splits", 1, MAX_ROWS, MAX_ROWS, 2),
                ("fwd_few", 1, MAX_ROWS, 4096, 64), ("fwd_few", 1, 32, MAX_ROWS, 64)]) == [(1,), (1,), (0,), (1,)]
    (p,), = ask([("bwd_splits", 1, 128, MAX_ROWS, 2)])
    assert 2 <= p <= 256


def test_parts_fit_the_chip_and_their_place():
    """All parts' workgroups fit 256 CUs at once, and a part has at least four tiles."""
    rng = random.Random(7)
    cases = [(rng.randint(1, 300), rng.randint(1, 20000), rng.randint(1, 20000), rng.choice([2, 4])) for _ in range(400)]
    for (heads, fixed, streamed, _), (p,) in zip(cases, ask([("bwd_splits", *c) for c in cases])):
        assert p == 1 or (p * heads * -(-fixed // 128) <= 256 and 4 * p <= -(-streamed // 64))


@pytest.mark.parametrize("R", [2 ** 28, 2 ** 29 - 1, 2 ** 29, 2 ** 30, MAX_ROWS - 255])
def test_linear_tiles_fit_one_launch(R):
    """The 128 and 64 tiles take a workgroup of 256 threads each, and a launch has at most 2^32 - 1 threads: calls with more
    small tiles than that go to the persistent 256-row shapes (y: 2 x R x F, grad x: 2 x R x K)."""
    for K, F in ((32, 32), (32, 96), (64, 32), (96, 64), (192, 32)):
        (y, gx, _, _), = ask([("linear", R, K, F)])
        for shape, width in ((y, F), (gx, K)):
            if shape >= 2:
                tile = 128 if shape == 2 else 64
                tiles = 2 * -(-R // tile) * -(-width // tile)
                assert -(-tiles // 8) * 8 * 256 < 2 ** 32, (R, K, F, shape)


# R, K, F and the measured times (us, graphs of calls back to back) of the 256, 192, 128 and 64 tiles: the forward, and a whole
# backward without bias whose grad x takes the shape
MEASURED_FORWARD = [
    (2048, 768, 1536, (21.4, 18.5, 21.2, 21.6)), (4096, 1152, 768, (25.7, 22.1, 26.0, 25.4)),
    (4096, 768, 768, (19.6, 17.0, 19.5, 18.8)), (2048, 384, 1536, (13.7, 12.2, 13.9, 14.2)),
    (8192, 384, 384, (13.3, 11.6, 13.8, 13.7)), (256, 4608, 1152, (72.5, 58.0, 38.0, 18.8)),
    (1024, 1536, 1152, (29.5, 24.2, 17.0, 17.3)), (2048, 1152, 3456, (32.8, 41.8, 53.7, 58.1)),
    (16384, 384, 1152, (37.3, 33.0, 59.4, 70.5)), (500, 768, 768, (17.2, 14.1, 9.6, 5.6)),
    (64, 768, 768, (17.1, 14.1, 9.5, 5.3)), (65536, 32, 128, (14.9, 13.8, 17.9, 21.8)),
    (8192, 256, 32, (9.8, 8.2, 5.8, 3.8)), (16384, 64, 1152, (19.8, 18.4, 33.7, 42.9)),
    (2048, 64, 4608, (14.7, 12.6, 20.5, 23.9)), (8192, 64, 1152, (14.8, 12.6, 20.5, 23.4)),
    (8192, 4608, 1152, (181.6, 149.2, 211.0, 246.5)), (5000, 96, 1312, (11.9, 13.9, 18.5, 19.9)),
]
MEASURED_BACKWARD = [
    (4096, 768, 384, (34.5, 32.6, 35.2, 36.2)), (16384, 1152, 1152, (177.2, 164.2, 222.5, 244.0)),
    (8192, 96, 1536, (51.0, 44.8, 37.2, 35.3)), (500, 768, 768, (24.6, 21.0, 16.5, 12.2)),
    (2048, 768, 768, (36.2, 32.9, 29.5, 29.8)), (1024, 768, 1152, (34.8, 30.0, 23.7, 20.7)),
]


@pytest.mark.parametrize("R,K,F,times,which", [(*m, 0) for m in MEASURED_FORWARD] + [(*m, 1) for m in MEASURED_BACKWARD])
def test_linear_tiles_against_measured_times(R, K, F, times, which):
    """The chosen shape is the fastest measured one, or within 4 % of it."""
    shape = ask([("linear", R, K, F)])[0][which]
    assert times[shape] <= 1.04 * min(times), (shape, times)


# float32: heads, M, N, d and the measured times (us, graphs of calls back to back) of the plain-ALU and of the matrix-core kernels,
# forward and backward
MEASURED_F32 = [
    (1, 1, 1, 4, (3.3, 3.9), (8.4, 9.0)), (1, 1, 1, 64, (4.5, 4.8), (20.7, 12.3)),
    (1, 4, 4, 16, (3.9, 4.0), (12.0, 9.1)), (16384, 1, 1, 16, (28.8, 43.4), (103.5, 148.2)),
    (16384, 1, 1, 64, (64.9, 87.8), (303.3, 325.8)), (16384, 1, 1, 128, (126.2, 296.9), (590.2, 1042.8)),
    (16384, 4, 4, 128, (170.5, 317.5), (1022.6, 1223.8)), (16384, 4, 4, 32, (61.0, 60.6), (272.2, 169.7)),
    (2048, 4, 4, 64, (15.4, 12.8), (67.1, 44.3)), (2048, 1, 16, 128, (52.8, 42.9), (320.8, 146.0)),
    (2048, 16, 1, 64, (37.6, 14.9), (158.2, 52.9)), (1, 16, 1, 128, (7.3, 7.6), (45.5, 20.9)),
    (2048, 8, 8, 64, (34.2, 13.9), (196.7, 50.0)), (2048, 64, 4, 32, (111.7, 34.0), (419.0, 73.6)),
]


@pytest.mark.parametrize("heads,M,N,d,fwd,bwd", MEASURED_F32)
def test_f32_kernels_against_measured_times(heads, M, N, d, fwd, bwd):
    """The kernel family a float32 call takes is the faster measured one, or within 5 % of it; with gO alone always the matrix
    cores."""
    mfma_fwd, mfma_bwd, mfma_go = ask([("f32", heads, M, N, d)])[0]
    assert fwd[mfma_fwd] <= 1.05 * min(fwd)
    assert bwd[mfma_bwd] <= 1.05 * min(bwd)
    assert mfma_go == 1


def test_f32_kernels_of_ordinary_sizes():
    """More than eight rows on both sides: the matrix cores, for every head dim that they read and no other."""
    rng = random.Random(3)
    cases = [(rng.choice([1, 48, 5000, 20000]), rng.randint(9, 5000), rng.randint(17, 5000), rng.randint(1, 256)) for _ in range(200)]
    for (_, _, _, d), got in zip(cases, ask([("f32", *c) for c in cases])):
        assert got == ((1, 1, 1) if d % 4 == 0 and d <= 128 else (0, 0, 0))


# heads, rows, d and the measured whole backward (us) with results straight from the accumulators and as whole rows: gO alone;
# with the tangent and at most 64 rows on the other side
MEASURED_STORES = [
    (1, 33, 72, (9.4, 10.3)), (2048, 33, 72, (44.8, 47.9)), (64, 64, 72, (10.0, 10.8)), (1024, 64, 72, (31.9, 32.8)),
    (1024, 64, 64, (28.0, 26.7)), (2048, 64, 128, (93.5, 84.2)), (2048, 128, 8, (26.4, 28.0)), (16, 128, 64, (14.5, 13.1)),
    (16, 128, 72, (12.8, 13.1)), (256, 128, 72, (18.3, 16.8)), (2048, 128, 72, (102.8, 89.9)), (1, 128, 128, (22.0, 19.2)),
    (256, 512, 104, (142.4, 129.0)), (1, 512, 64, (28.8, 27.2)), (512, 256, 32, (32.4, 31.9)), (64, 33, 104, (12.5, 13.4)),
    (256, 96, 88, (16.3, 15.0)), (2048, 96, 48, (54.2, 50.6)), (1, 96, 56, (9.3, 9.7)),
]


MEASURED_STORES_TANGENT = [
    (64, 33, 104, (22.5, 25.7)), (1024, 64, 104, (116.8, 123.4)), (166, 976, 128, (179.4, 162.7)), (64, 64, 128, (30.6, 30.8)),
]


@pytest.mark.parametrize("tangent,heads,rows,d,times", [(0, *m) for m in MEASURED_STORES] + [(1, *m) for m in MEASURED_STORES_TANGENT])
def test_stores_of_the_generic_backward_against_measured_times(tangent, heads, rows, d, times):
    (whole,), = ask([("rows", tangent, heads, rows, d)])
    assert times[whole] <= 1.02 * min(times)


# ---------------------------------------------------------------- the sizes of the GPU tests are where they claim to be
@pytest.mark.parametrize("shape,tiles,parts", dc.LINEAR)
def test_linear_cases(shape, tiles, parts):
    R, K, F = shape
    (y, gx, gw, splits), = ask([("linear", *shape)])
    assert tuple((256, 192, 128, 64)[c] for c in (y, gx, gw)) == tiles
    assert (splits > 1 or gw < 2) == parts   # (the 128 and 64 tiles of one split write gW themselves)


def test_linear_cases_are_ragged_everywhere():
    for product, contraction, column in (("y", 1, 2), ("gx", 2, 1), ("gw", 0, 1)):
        for tile in (256, 192, 128, 64):
            assert any(t[("y", "gx", "gw").index(product)] == tile and s[contraction] % 64 != 0 and s[column] % tile != 0 and s[column] > tile
                       for s, t, _ in dc.LINEAR), (product, tile)


def test_forward_cases():
    eight = [(c, d) for c in dc.FORWARD_EIGHT_WAVES for d in dc.FORWARD_EIGHT_WAVES_DIMS]
    four = [(c, d) for c in dc.FORWARD_FOUR_WAVES for d in dc.FORWARD_FOUR_WAVES_DIMS]
    four += [(c, d) for c in dc.FORWARD_FOUR_WAVES_WIDE for d in (104, 128)]
    for cases in (eight, four):
        assert set(ask([("fwd_few", *c, d) for c, d in cases])) == {(0,)}
    assert all(M > 128 and N >= 512 and d <= 96 for (_, M, N), d in eight)
    assert all(N >= 128 and (N < 512 or M <= 128 or d > 96) for (_, M, N), d in four)
    assert [bool(a) for a, in ask([("fwd_few", *c[:4]) for c in dc.FORWARD_LINES])] == [c[4] for c in dc.FORWARD_LINES]


@pytest.mark.parametrize("B,T,C,dtype", dc.GATE_MANY_ROWS)
def test_gate_cases(B, T, C, dtype):
    if not os.path.exists(binding.LIB_PATH):
        tvm_build.build()
    need = binding.lib().tvmattn_gate_jvp_bwd_workspace_bytes(B, T, C, {"f32": binding.TVMATTN_F32, "bf16": binding.TVMATTN_BF16}[dtype])
    assert need > 32 * B * 2 * C * 4 + 255
