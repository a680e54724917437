"""The rules that choose kernels and cut work, evaluated on the host (tests/dispatch_rules.py)."""
import random

import pytest

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
