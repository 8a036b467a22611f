"""The contractions in every tile they are cut into (gemm_xs_kernel's four and gemm_xb_kernel's), each
at sizes that its dispatch rule sends there and that end inside tiles, K-tiles and K-quads: the whole
oracle, from a workspace of NaN bytes, with the bars of test_gpu_parity.py."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from test_gpu_parity import TOL, _check_full, _nan_workspace, _to_dev, lce  # noqa: F401

pytestmark = pytest.mark.gpu

# (N, H, V, dtype, chunk_tokens)
STEPS = [
    (33, 72, 32077, "bf16", 0),       # logits 128 x 64, per-chunk K check
    (64, 192, 32000, "fp16", 0),      # the same, whole K-tiles
    (65, 40, 2081, "bf16", 0),        # 64 x 64 everywhere, K ends inside a K-tile
    (191, 136, 4127, "fp16", 0),
    (100, 36, 1061, "fp32", 0),       # fp32 K-quads of 16 ids: V = 16 q + 5
    (300, 264, 33003, "bf16", 300),   # logits and dW 128 x 256
    (511, 328, 20001, "fp16", 511),
    (700, 260, 9001, "fp32", 700),    # fp32 128 x 256
    (520, 1032, 9007, "bf16", 520),   # dH 256 x 256 by eight waves, split
    (1100, 520, 9000, "bf16", 1100),  # dH by gemm_xb_kernel, split
    (1200, 264, 12000, "bf16", 448),  # dW 128 x 256 added to across chunks
    (1200, 264, 12000, "fp16", 448),
    (640, 264, 12000, "bf16", 64),    # and across more than the carry limit, in fp32
    (300, 2056, 32700, "bf16", 300),  # logits by gemm_xb_kernel (H >= 3 N)
    (4100, 8200, 1000, "bf16", 4100),  # dW 256 x 256 by eight waves
    (4100, 136, 65600, "bf16", 4100),  # dW by gemm_xb_kernel (one column of tiles)
]


@pytest.mark.parametrize("N,H,V,dtype,chunk", STEPS)
def test_step_in_every_tile(lce, N, H, V, dtype, chunk):  # noqa: F811
    d = workloads.make_inputs("llama3_8b", seed=31, N=N, H=H, V=V, dtype=dtype)
    _check_full(lce, d, chunk_tokens=chunk, workspace=_nan_workspace(lce, d, chunk))


# Forward only: slice maxima in every slice height (32, 128 rows), tokens up to a tile's edge.
@pytest.mark.parametrize("N,H,V,dtype", [(1, 72, 32001, "bf16"), (64, 64, 40000, "fp16"), (65, 72, 3001, "bf16"),
                                         (63, 36, 1999, "fp32"), (257, 264, 33001, "bf16"), (500, 100, 9000, "fp32")])
def test_forward_in_every_tile(lce, N, H, V, dtype):  # noqa: F811
    d = workloads.make_inputs("llama3_8b", seed=32, N=N, H=H, V=V, dtype=dtype)
    print(f"case forward {N}x{H}x{V} {dtype}", flush=True)
    X, W, y = _to_dev(d)
    loss, lse = lce.forward(X, W, y, d["ignore_index"], "none", return_lse=True)
    ref = oracle.forward(d["hidden"], d["weight"], d["labels"], d["ignore_index"], "none")
    # fp32 sums of H products and V exponentials; the bars of the reduced loss hold for every token.
    assert np.abs(loss.cpu().numpy() - ref["loss"]).max() <= TOL[dtype][0] * np.abs(ref["loss"]).max()
    assert np.abs(lse.cpu().numpy() - ref["lse"]).max() <= TOL[dtype][0] * np.abs(ref["lse"]).max()


@pytest.mark.parametrize("N,H,V,lo,hi", [(65, 72, 3001, 0, 40), (65, 72, 3001, 64, 96), (64, 64, 40000, 128, 256)])
def test_forward_with_slices_of_minus_inf(lce, N, H, V, lo, hi):  # noqa: F811
    """Ids whose logits are -inf add nothing to a token's sum, also where they fill a whole partial (64 x 64 and
    128 x 64 tiles: 32 and 128 ids): the other ids' losses, of the oracle without them."""
    d = workloads.make_inputs("llama3_8b", seed=33, N=N, H=H, V=V, dtype="bf16")
    hidden = d["hidden"].abs() + 0.01
    weight, labels = d["weight"].clone(), torch.arange(N) + hi
    ref = oracle.forward(hidden, torch.cat((weight[:lo], weight[hi:])), labels - (hi - lo), -100, "none")
    weight[lo:hi] = -float("inf")
    loss, lse = lce.forward(hidden.cuda(), weight.cuda(), labels.cuda(), -100, "none", return_lse=True)
    assert np.abs(loss.cpu().numpy() - ref["loss"]).max() <= TOL["bf16"][0] * np.abs(ref["loss"]).max()
    assert np.abs(lse.cpu().numpy() - ref["lse"]).max() <= TOL["bf16"][0] * np.abs(ref["lse"]).max()
