"""The autograd wrappers' backward: the gradients times the upstream one, by the library's kernel for plain
tensors and by torch's operators for the rest (batched or differentiable upstream gradients)."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu

DT = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}


@pytest.fixture(scope="module")
def lce():
    import paper_2603_16428_amd as m
    m.load_library()
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return m


def _leaves(lce, dtype, N=70, H=72, V=1031):
    d = workloads.random_case(N, H, V, dtype=dtype, seed=5, w_std=0.5)
    X, W = (d[k].cuda().requires_grad_() for k in ("hidden", "weight"))
    return X, W, d["labels"].cuda()


@pytest.mark.parametrize("dtype", list(DT))
@pytest.mark.parametrize("factor", [1.0, 0.37, -3e4])
def test_scaled_gradients(lce, dtype, factor):
    X, W, y = _leaves(lce, dtype)
    _, dH, dW = lce.forward_backward(X.detach(), W.detach(), y)
    loss = lce.linear_cross_entropy(X, W, y)
    (loss * factor).backward(retain_graph=True)
    first = X.grad.clone(), W.grad.clone()
    for got, g in zip(first, (dH, dW)):  # one fp32 product, rounded once
        assert torch.equal(got, (g.float() * factor).to(g.dtype))
    X.grad = W.grad = None
    (loss * factor).backward()           # the saved gradients are as they were
    assert torch.equal(X.grad, first[0]) and torch.equal(W.grad, first[1])


# Sizes around a thread's 16 bytes, a block's 16 KB and the boundaries between the jobs of one launch.
@pytest.mark.parametrize("dtype", list(DT))
@pytest.mark.parametrize("sizes", [(1,), (7, 8, 9), (4096, 8191, 8193), (16385, 3, 100000)])
def test_scale_sizes(lce, dtype, sizes):
    from paper_2603_16428_amd.lce import _scaled
    gen = torch.Generator().manual_seed(1)
    ts = [torch.randn(n, generator=gen).to(DT[dtype]).cuda() for n in sizes]
    f = torch.tensor(0.3, device="cuda")
    for got, t in zip(_scaled(f, ts), ts):
        assert torch.equal(got, (t.float() * f).to(t.dtype))


def test_other_upstream_gradients(lce):
    X, W, y = _leaves(lce, "bf16")
    loss = lce.linear_cross_entropy(X, W, y)
    one = torch.autograd.grad(loss, (X, W), retain_graph=True)
    ones = torch.ones(3, device="cuda")
    for got, want in zip(torch.autograd.grad(loss, (X, W), ones, retain_graph=True, is_grads_batched=True), one):
        assert got.shape == (3, *want.shape) and all(torch.equal(got[k], want) for k in range(3))
    scale = torch.tensor(2.0, device="cuda", requires_grad=True)
    gX, = torch.autograd.grad(loss * scale, X, create_graph=True)
    back, = torch.autograd.grad(gX.float().sum(), scale)
    assert torch.isfinite(back) and abs(back.item() - one[0].float().sum().item()) <= 1e-2 * one[0].float().abs().sum().item()


def test_lazily_negated_and_zero_gradients(lce):
    """A negative bit (the imaginary part of a conjugate) and a zero tensor have other values than the
    memory that their pointers name, as upstream gradients and as tensors that a saved-tensor hook gives."""
    X, W, y = _leaves(lce, "bf16")
    loss = lce.linear_cross_entropy(X, W, y)
    want = torch.autograd.grad(loss, (X, W), torch.tensor(-2.0, device="cuda"), retain_graph=True)
    neg = torch.complex(torch.tensor(0.0), torch.tensor(2.0)).cuda().conj().imag
    assert neg.is_neg() and neg.item() == -2.0
    for got, w in zip(torch.autograd.grad(loss, (X, W), neg, retain_graph=True), want):
        assert torch.equal(got, w)
    zero = torch._efficientzerotensor((), device="cuda")
    for got in torch.autograd.grad(loss, (X, W), zero, retain_graph=True):
        assert not got.any()
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, torch._neg_view):
        hooked = lce.linear_cross_entropy(X, W, y)
    for got, w in zip(torch.autograd.grad(hooked, (X, W), torch.tensor(2.0, device="cuda")), want):
        assert torch.equal(got, w)


def test_rmsnorm_wrapper(lce):
    d = workloads.make_rmsnorm_inputs("llama3_8b", seed=3, N=70, H=72, V=1031)
    h, g, W = (d[k].cuda().requires_grad_() for k in ("hidden", "gamma", "weight"))
    y = d["labels"].cuda()
    _, *grads = lce.rmsnorm_forward_backward(h.detach(), g.detach(), W.detach(), y, d["eps"])
    (lce.rmsnorm_linear_cross_entropy(h, g, W, y, d["eps"]) * 0.5).backward()
    for t, want in zip((h, g, W), grads):
        assert torch.equal(t.grad, (want.float() * 0.5).to(want.dtype))
