"""The contractions in every tile they are cut into (gemm_xs_kernel's four and gemm_xb_kernel's), each
at sizes that its dispatch rule sends there and that end inside tiles, K-tiles and K-quads: the whole
oracle, from a workspace of NaN bytes, with the bars of test_gpu_parity.py."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_2603_16428_amd.lce import _plan_tiles
from test_gpu_parity import TOL, _check_full, _nan_workspace, _to_dev, lce  # noqa: F401

pytestmark = pytest.mark.gpu

DTYPES = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}

# (N, H, V, dtype, chunk_tokens, tiles of logits, dH and dW). test_tile_routes.py checks the tiles without a GPU.
STEPS = [
    (33, 72, 32077, "bf16", 0, "128x64 64 128"),       # logits of up to 64 tokens, per-chunk K check
    (64, 192, 32000, "fp16", 0, "128x64 64 128"),      # the same, whole K-tiles
    (65, 40, 2081, "bf16", 0, "64 64 64"),             # K ends inside a K-tile; dW added to across chunks
    (191, 136, 4127, "fp16", 0, "64 64 64"),
    (100, 36, 1061, "fp32", 0, "64 64 64"),            # fp32 K-quads of 16 ids: V = 16 q + 5
    (300, 264, 33003, "bf16", 300, "128 64 128"),
    (511, 328, 20001, "fp16", 511, "128 128 128"),
    (700, 260, 9001, "fp32", 700, "128 64 64"),        # fp32 128 x 256
    (1000, 1024, 20003, "fp32", 1000, "128 128 128"),  # the same, whole K-tiles
    (1000, 1024, 20003, "fp32", 512, "64 128 128"),    # fp32 dW added to across chunks
    (520, 1032, 9007, "bf16", 520, "128 128 128"),     # dH split
    (1100, 520, 9000, "bf16", 1100, "128 128 128"),
    (1100, 2056, 20007, "bf16", 1100, "128 256 128"),  # dH 256 x 256 by eight waves, split
    (2100, 1048, 9007, "fp16", 2100, "128 256 128"),
    (2100, 136, 100003, "bf16", 2100, "128 xb 128"),   # dH by gemm_xb_kernel, split
    (2100, 136, 100003, "fp16", 2100, "128 xb 128"),
    (1200, 264, 12000, "bf16", 448, "256 64 128"),     # dW 128 x 256 added to across chunks
    (1200, 264, 12000, "fp16", 448, "256 64 128"),
    (1200, 256, 12000, "bf16", 448, "256 64 64"),      # logits 256 x 256 by eight waves, whole K-tiles
    (640, 264, 12000, "bf16", 64, "64 64 128"),        # more chunks than the carry limit, in fp32
    (520, 5128, 20003, "bf16", 0, "xb 256 128"),       # logits by gemm_xb_kernel, per-chunk K check
    (520, 5128, 20003, "fp16", 0, "xb 256 128"),
    (1000, 4096, 16003, "bf16", 0, "xb 128 128"),      # the same, whole K-tiles
    (520, 5184, 20003, "fp16", 0, "xb 256 128"),
    (4100, 8200, 1000, "bf16", 4100, "128 256 256"),   # dW 256 x 256 by eight waves
    (4300, 8200, 1000, "bf16", 4160, "128 256 256"),   # and added to
    (4300, 8200, 1000, "fp16", 4160, "128 256 256"),
    (4100, 136, 65600, "bf16", 4100, "128 256 xb"),    # dW by gemm_xb_kernel (one column of tiles)
    (4300, 136, 65600, "fp16", 4160, "128 256 xb"),    # and added to
]


@pytest.mark.parametrize("N,H,V,dtype,chunk,tiles", STEPS)
def test_step_in_every_tile(lce, N, H, V, dtype, chunk, tiles):  # noqa: F811
    assert _plan_tiles(N, H, V, DTYPES[dtype], True, chunk) == tuple(tiles.split())
    d = workloads.make_inputs("llama3_8b", seed=31, N=N, H=H, V=V, dtype=dtype)
    _check_full(lce, d, chunk_tokens=chunk, workspace=_nan_workspace(lce, d, chunk))


# Forward only: slice maxima in every slice height (32 and 128 rows), tokens up to a tile's edge.
FORWARD = [
    (1, 72, 32001, "bf16", "128x64"),
    (64, 64, 40000, "fp16", "128x64"),
    (65, 72, 3001, "bf16", "64"),
    (63, 36, 1999, "fp32", "64"),
    (191, 136, 4127, "fp16", "64"),
    (257, 264, 33001, "bf16", "128"),
    (300, 256, 20001, "fp16", "128"),
    (500, 100, 9000, "fp32", "128"),
    (69, 288, 25521, "bf16", "256"),
    (70, 256, 26001, "fp16", "256"),
    (520, 5128, 20003, "bf16", "xb"),
    (257, 5128, 30003, "fp16", "xb"),
    (257, 5120, 20003, "fp16", "xb"),
    (400, 4096, 20003, "bf16", "xb"),
]


@pytest.mark.parametrize("N,H,V,dtype,tile", FORWARD)
def test_forward_in_every_tile(lce, N, H, V, dtype, tile):  # noqa: F811
    assert _plan_tiles(N, H, V, DTYPES[dtype], False) == (tile, None, None)
    d = workloads.make_inputs("llama3_8b", seed=32, N=N, H=H, V=V, dtype=dtype)
    print(f"case forward {N}x{H}x{V} {dtype}", flush=True)
    X, W, y = _to_dev(d)
    loss, lse = lce.forward(X, W, y, d["ignore_index"], "none", return_lse=True)
    ref = oracle.forward(d["hidden"], d["weight"], d["labels"], d["ignore_index"], "none")
    # fp32 sums of H products and V exponentials; the bars of the reduced loss hold for every token.
    assert np.abs(loss.cpu().numpy() - ref["loss"]).max() <= TOL[dtype][0] * np.abs(ref["loss"]).max()
    assert np.abs(lse.cpu().numpy() - ref["lse"]).max() <= TOL[dtype][0] * np.abs(ref["lse"]).max()


@pytest.mark.parametrize("N,H,V,lo,hi,tile", [
    (65, 72, 3001, 0, 40, "64"), (65, 72, 3001, 64, 96, "64"), (64, 64, 40000, 128, 256, "128x64"),
    (257, 264, 33001, 256, 400, "128"), (69, 288, 25521, 128, 256, "256"), (400, 4096, 20003, 128, 256, "xb"),
    (257, 5128, 30003, 0, 256, "xb")])
def test_forward_with_slices_of_minus_inf(lce, N, H, V, lo, hi, tile):  # noqa: F811
    """Ids whose logits are -inf add nothing to a token's sum, also where they fill a whole partial (32 or 128
    ids, by the tile): the other ids' losses, of the oracle without them."""
    assert _plan_tiles(N, H, V, torch.bfloat16, False)[0] == tile
    d = workloads.make_inputs("llama3_8b", seed=33, N=N, H=H, V=V, dtype="bf16")
    hidden = d["hidden"].abs() + 0.01
    weight, labels = d["weight"].clone(), torch.arange(N) + hi
    ref = oracle.forward(hidden, torch.cat((weight[:lo], weight[hi:])), labels - (hi - lo), -100, "none")
    weight[lo:hi] = -float("inf")
    loss, lse = lce.forward(hidden.cuda(), weight.cuda(), labels.cuda(), -100, "none", return_lse=True)
    assert np.abs(loss.cpu().numpy() - ref["loss"]).max() <= TOL["bf16"][0] * np.abs(ref["loss"]).max()
    assert np.abs(lse.cpu().numpy() - ref["lse"]).max() <= TOL["bf16"][0] * np.abs(ref["lse"]).max()
