"""The rows of test_gpu_tiles.py reach the tiles that they name, and every tile that automatic plans choose
is among them (no GPU: the library's own plans)."""
import random

import pytest

from paper_2603_16428_amd.lce import _plan_tiles
from test_auto_chunk import _log_uniform
from test_gpu_tiles import DTYPES, FORWARD, STEPS


@pytest.mark.parametrize("N,H,V,dtype,chunk,tiles", STEPS)
def test_steps(N, H, V, dtype, chunk, tiles):
    assert _plan_tiles(N, H, V, DTYPES[dtype], True, chunk) == tuple(tiles.split())


@pytest.mark.parametrize("N,H,V,dtype,tile", FORWARD)
def test_forward(N, H, V, dtype, tile):
    assert _plan_tiles(N, H, V, DTYPES[dtype], False) == (tile, None, None)


def test_every_tile_has_a_row():
    rows = {(c, dtype, t) for _, _, _, dtype, _, tiles in STEPS for c, t in zip(("logits", "dH", "dW"), tiles.split())}
    rows |= {("forward", dtype, t) for _, _, _, dtype, t in FORWARD}
    rng = random.Random(11)
    for _ in range(4000):
        N, H, V = (_log_uniform(rng, *r) for r in ((1, 16384), (1, 1536), (64, 152064)))
        for dtype, dt in DTYPES.items():
            seen = {(c, dtype, t) for c, t in zip(("logits", "dH", "dW"), _plan_tiles(N, 8 * H, V, dt))}
            seen.add(("forward", dtype, _plan_tiles(N, 8 * H, V, dt, False)[0]))
            assert seen <= rows, (N, 8 * H, V, dtype, seen - rows)
