"""The automatic chunk of a training call, by the library's own plan (no GPU): few tokens are one chunk,
more make chunks that cover them without a last one of a few tokens, and e stays within its bound."""
import math
import random

import pytest
import torch

from paper_2603_16428_amd import lce

DTYPES = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}


@pytest.mark.parametrize("N,H,dtype,chunk", [
    (1, 64, "bf16", 1), (1000, 4096, "bf16", 1000), (2048, 2048, "bf16", 2048), (2048, 4096, "fp16", 2048),
    (2049, 4096, "bf16", 1088), (3000, 4096, "bf16", 1536), (256, 256, "fp32", 256), (257, 256, "fp32", 192),
    (129, 8, "bf16", 64), (1000, 768, "bf16", 512), (4096, 768, "bf16", 1024), (8192, 4096, "bf16", 4096)])
def test_auto_chunk(N, H, dtype, chunk):
    dt = DTYPES[dtype]
    assert lce.auto_chunk_tokens(N, H, 5000, dt) == chunk
    info = lce.plan_info(N, H, 5000, dt)
    assert info["chunk_tokens"] == chunk and info["chunks"] == -(-N // chunk)
    # e is no larger than W (twice W where that avoids the fp32 carry), but for the 64-token minimum.
    assert chunk <= max(64, H, 2 * H if -(-N // H) > 4 and dtype == "bf16" else 0)


def _log_uniform(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def _fp32_chunk(N, H):
    """Half of the tokens rounded down to 64, at most H: what an fp32 call's sums are sized for."""
    return min(N, max(64, min(H, -(-N // 2)) // 64 * 64))


def _fp32_splits(N, H):
    """The splits (1 to 8) that fill 256 CUs best with 256 x 256 tiles of such a chunk."""
    tiles = -(-_fp32_chunk(N, H) // 256) * -(-H // 256)
    return min(range(1, 9), key=lambda s: (round(-(-tiles * s // 256) / s + (0.03 * s if s > 1 else 0), 9), s))


# The last three: N / 2 rounded up to 64 is one row of tiles more than rounded down.
@pytest.mark.parametrize("N,H,V", [(512, 512, 20000), (2000, 2048, 8000), (1024, 4096, 4096), (4096, 2048, 8192),
                                   (11786, 7896, 12703), (10287, 5664, 9125), (9269, 6248, 13225)])
def test_fp32_dh_splits(N, H, V):
    """fp32: a dH entry's running sum is no longer than with the splits that fill 256 CUs with 256 x 256
    tiles of half the tokens, whatever the chunk."""
    assert lce.plan_info(N, H, V, torch.float32)["dh_splits"] >= _fp32_splits(N, H)


def test_fp32_dh_splits_over_the_range():
    rng = random.Random(7)
    for _ in range(2000):
        N, H, V = (_log_uniform(rng, *r) for r in ((64, 16384), (32, 1536), (4096, 152064)))
        assert lce.plan_info(N, 8 * H, V, torch.float32)["dh_splits"] >= _fp32_splits(N, 8 * H), (N, 8 * H, V)


@pytest.mark.parametrize("N,H,V,dtype,chunk", [
    (1652, 1159040, 60913, "bf16", 768), (380, 1958364, 56, "fp32", 128), (625, 3319736, 7, "fp16", 256),
    (1100, 1048576, 1000, "bf16", 512), (65, 4000000, 5, "bf16", 65)])
def test_wide_rows_are_accepted(N, H, V, dtype, chunk):
    """Rows so wide that one chunk's blocked copies would pass 2^31 bytes: chunks of half the tokens."""
    dt = DTYPES[dtype]
    assert lce.plan_info(N, H, V, dt)["chunk_tokens"] == chunk
    assert lce.workspace_size(N, H, V, dt) > 0


def test_wide_rows_are_accepted_forward_only():
    """More than 16384 tokens in chunks of half of them, where the half rounded up would not fit the limit."""
    info = lce.plan_info(40068, 26744, 56849, torch.float32, with_backward=False)
    assert info["chunk_tokens"] == 20032 and info["chunks"] == 3


def test_dh_partials_stay_within_their_bound():
    """dH's fp32 partials: below W (or 64 MB) with automatic chunks; below the chunk's e, or in eight splits,
    with the caller's chunk, so that a small one keeps the workspace small."""
    rng = random.Random(13)
    cases = [(203, 5472, 135757, "fp32", 0), (8192, 4096, 128256, "bf16", 64), (4096, 768, 50257, "bf16", 64)]
    for _ in range(2000):
        N, H, V = (_log_uniform(rng, *r) for r in ((64, 16384), (32, 1536), (64, 152064)))
        cases.append((N, 8 * H, V, rng.choice(tuple(DTYPES)), rng.choice((0, 64, 64 * rng.randint(1, 64)))))
    for N, H, V, dtype, chunk in cases:
        size = 4 if dtype == "fp32" else 2
        info = lce.plan_info(N, H, V, DTYPES[dtype], True, chunk)
        if info["dh_splits"] == 1:
            continue
        tokens = info["chunk_tokens"]
        part, eight = info["dh_splits"] * tokens * H * 4, 8 * tokens * H * 4
        e = -(-tokens // 64) * 64 * -(-V // 256) * 256 * size
        bound = max(e, eight) if chunk else max(64 << 20, V * H * size, eight if dtype == "fp32" else 0)
        assert part <= bound, (N, H, V, dtype, chunk)
