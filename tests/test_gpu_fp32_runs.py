"""fp32 dW: the running sums of an automatic call are no longer than those of a call in chunks of half the
tokens (rounded down to 64, at most H), whose dW it adds up the same way, so its error against float64 is
no larger."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from test_auto_chunk import _fp32_chunk
from test_gpu_parity import _check_full, _nan_workspace, _to_dev, lce  # noqa: F401

pytestmark = pytest.mark.gpu


# One chunk in 2, 4, 3 and 3 runs (64 x 64 tiles, the last two 128 x 256 tiles), two chunks of 1536 tokens in
# two runs each, and one with a last run of one token.
@pytest.mark.parametrize("N,H,V", [(256, 256, 4096), (252, 352, 6001), (1000, 1024, 5000), (2000, 2048, 4104),
                                   (3000, 2048, 4097), (129, 256, 1031)])
def test_dw_error_of_one_chunk(lce, N, H, V):  # noqa: F811
    d = workloads.make_inputs("llama3_8b", seed=41, N=N, H=H, V=V, dtype="fp32")
    print(f"case {N}x{H}x{V} fp32", flush=True)
    X, W, y = _to_dev(d)
    ref = oracle.forward_backward(d["hidden"], d["weight"], d["labels"], d["ignore_index"], d["reduction"])
    err = [np.linalg.norm(lce.forward_backward(X, W, y, d["ignore_index"], d["reduction"], chunk_tokens=c)[2]
                          .cpu().numpy() - ref["dW"]) for c in (0, _fp32_chunk(N, H))]
    print(f"  dW off by {err[0]:.4g}, in chunks by {err[1]:.4g}", flush=True)
    # The same sums, but for the rounding of the tokens' factors: their errors are alike to a few percent (runs
    # twice as long: 1.4 times).
    assert err[0] <= 1.1 * err[1]
    _check_full(lce, d, chunk_tokens=0, workspace=_nan_workspace(lce, d, 0), ref=ref)
