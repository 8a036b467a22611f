"""The calls that the output-layer step is timed on: what each stands for, its inputs, its float64 result.

A case is one call (`kind`) at N tokens, hidden size H and V vocabulary ids, in `dtype`:

  forward   lce.forward: per-token losses and log-sum-exps ("none") or the reduced loss (evaluation)
  train     lce.forward_backward with the workspace and the outputs a training program keeps
  autograd  lce.linear_cross_entropy(...).backward() on leaf tensors
  rmsnorm   lce.rmsnorm_forward_backward: the final RMSNorm in front of the step
  head      lce.head_train_step: one optimizer step of the layer, weights and Adam states on the host

Inputs follow `workloads` (unit-RMS hidden rows or N(0,1) 4/sqrt(H), W ~ w_std N(0,1), Zipf or uniform
labels, a share of ignored tokens), drawn on the GPU from the seed.
"""
import math

import torch

import paper_2603_16428_amd as lce

IGNORE = -100
DTYPES = {"bf16": torch.bfloat16, "fp16": torch.float16, "fp32": torch.float32}
LR, BETAS, ADAM_EPS = 1e-4, (0.9, 0.999), 1e-8
RMS_EPS = 1e-5


def _case(name, kind, N, H, V, dtype="bf16", reduction="mean", ignore=0.1, w_std=0.02, zipf=1.1):
    return {"name": name, "kind": kind, "N": N, "H": H, "V": V, "dtype": dtype, "reduction": reduction,
            "ignore": ignore, "w_std": w_std, "zipf": zipf}


def listed():
    return [
        # Scoring one short prompt with a Llama-3-8B head: the smallest call of a serving program.
        _case("score_prompt", "forward", 24, 4096, 128256, reduction="none", ignore=0.0),
        # Perplexity of a batch of 8 x 1024 tokens, no gradients, token by token.
        _case("eval_llama", "forward", 8192, 4096, 128256, reduction="none"),
        # The smallest training workload of the repository: float32, everything a few microseconds' work.
        _case("train_tiny_fp32", "train", 256, 256, 4096, "fp32", ignore=0.05, zipf=0.0),
        # One ragged sequence per step (batch 1, not padded) on a Llama-3-8B head.
        _case("train_one_sequence", "train", 1000, 4096, 128256),
        # GPT-2 small: short rows, an odd vocabulary, 4 x 1024 tokens.
        _case("train_gpt2", "train", 4096, 768, 50257),
        # The repository's small workload through autograd, as a training loop calls it.
        _case("autograd_small", "autograd", 2048, 2048, 32000),
        # The same sizes in float16, whose exponent range needs its own path for the gradient.
        _case("train_small_fp16", "train", 2048, 2048, 32000, "fp16"),
        # The final norm fused in front, 2 x 1024 tokens on a Llama-3-8B head.
        _case("rmsnorm_llama", "rmsnorm", 2048, 4096, 128256),
        # The headline workload: Llama-3-8B, 8 x 1024 tokens.
        _case("train_llama", "train", 8192, 4096, 128256),
        # Wide rows and a narrow vocabulary: Mistral-Large, 4 x 1024 tokens.
        _case("train_mistral", "train", 4096, 12288, 32768, ignore=0.05, w_std=0.01, zipf=0.0),
        # The largest: Qwen2.5-7B, 16 x 1024 tokens, summed loss, masked prompts.
        _case("train_qwen", "train", 16384, 3584, 152064, reduction="sum", ignore=0.15, zipf=1.05),
        # An optimizer step of a small head whose master weights live in host memory.
        _case("head_step", "head", 2048, 1024, 32000),
    ]


def _cost(c):
    # Time grows with the flops, and the float32 matrix unit is a sixteenth as fast as the 16-bit ones.
    flops = (2 if c["kind"] == "forward" else 6) * c["N"] * c["H"] * c["V"]
    return flops * (16 if c["dtype"] == "fp32" else 1)


def draw(rng):
    top = max(_cost(c) for c in listed())

    def log_uniform(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choices(("train", "forward", "autograd", "rmsnorm", "head"), (40, 25, 15, 15, 5))[0]
        dtype = rng.choices(("bf16", "fp16", "fp32"), (65, 20, 15))[0]
        N = log_uniform(1 if kind == "forward" else 64, 16384)
        H = 8 * log_uniform(32, 1536)
        V = log_uniform(4096, 152064)
        if kind == "head":
            N, H, V, dtype = min(N, 4096), min(H, 1024), min(V, 32000), "fp16" if dtype == "fp16" else "bf16"
        reduction = rng.choice(("none", "mean", "sum")) if kind == "forward" else rng.choice(("mean", "mean", "sum"))
        c = _case("", kind, N, H, V, dtype, reduction, ignore=rng.choice((0.0, 0.05, 0.1, 0.3)),
                  zipf=rng.choice((0.0, 1.05, 1.1)))
        del c["name"]
        if _cost(c) <= top and H * V <= 3584 * 152064:
            return c


def _inputs(case, seed):
    N, H, V, dtype = case["N"], case["H"], case["V"], DTYPES[case["dtype"]]
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    hidden = torch.randn((N, H), generator=g, device=dev)
    if case["kind"] == "rmsnorm":  # rows before the norm: the residual stream's size varies by token
        hidden *= torch.exp(math.log(0.25) + math.log(64.0) * torch.rand((N, 1), generator=g, device=dev))
    elif H <= 2048:
        hidden *= 4.0 / math.sqrt(H)
    else:
        hidden /= hidden.square().mean(1, keepdim=True).sqrt()
    weight = torch.empty((V, H), dtype=dtype, device=dev)
    for r in range(0, V, 16384):  # in blocks, so that the float32 draws stay small
        n = min(16384, V - r)
        weight[r:r + n] = case["w_std"] * torch.randn((n, H), generator=g, device=dev)
    if case["zipf"]:
        p = torch.arange(1, V + 1, device=dev, dtype=torch.float64) ** -case["zipf"]
        u = torch.rand(N, generator=g, device=dev, dtype=torch.float64)
        labels = torch.searchsorted(torch.cumsum(p, 0) / p.sum(), u).clamp_(max=V - 1)
    else:
        labels = torch.randint(0, V, (N,), generator=g, device=dev)
    labels[torch.randperm(N, generator=g, device=dev)[:int(round(case["ignore"] * N))]] = IGNORE
    gamma = (1.0 + 0.1 * torch.randn(H, generator=g, device=dev)).to(dtype)
    return hidden.to(dtype), weight, labels, gamma


def prepare(case, seed):
    hidden, weight, labels, gamma = _inputs(case, seed)
    N, H, V, dtype, kind = case["N"], case["H"], case["V"], DTYPES[case["dtype"]], case["kind"]
    s = {"kind": kind, "hidden": hidden, "weight": weight, "labels": labels, "reduction": case["reduction"]}
    dev = hidden.device
    if kind == "train":
        s["workspace"] = torch.empty(lce.workspace_size(N, H, V, dtype), dtype=torch.uint8, device=dev)
        s["out"] = (torch.empty(1, dtype=torch.float32, device=dev), torch.empty_like(hidden), torch.empty_like(weight))
    elif kind == "autograd":
        hidden.requires_grad_()
        weight.requires_grad_()
    elif kind == "rmsnorm":
        s["gamma"] = gamma
        s["workspace"] = torch.empty(lce.rmsnorm_workspace_size(N, H, V, dtype), dtype=torch.uint8, device=dev)
    elif kind == "head":
        s["head"] = lce.HeadState(weight)
        s["workspace"] = torch.empty(lce.workspace_size(N, H, V, dtype), dtype=torch.uint8, device=dev)
    return s


def run(s):
    kind, red = s["kind"], s["reduction"]
    if kind == "forward":
        return lce.forward(s["hidden"], s["weight"], s["labels"], IGNORE, red, return_lse=red == "none")
    if kind == "train":
        return lce.forward_backward(s["hidden"], s["weight"], s["labels"], IGNORE, red,
                                    workspace=s["workspace"], out=s["out"])
    if kind == "autograd":
        s["hidden"].grad = s["weight"].grad = None
        loss = lce.linear_cross_entropy(s["hidden"], s["weight"], s["labels"], IGNORE, red)
        loss.backward()
        return loss.detach(), s["hidden"].grad, s["weight"].grad
    if kind == "rmsnorm":
        return lce.rmsnorm_forward_backward(s["hidden"], s["gamma"], s["weight"], s["labels"], RMS_EPS, IGNORE, red,
                                            workspace=s["workspace"])
    head = s["head"]
    loss, grad_hidden, _ = lce.head_train_step(head, s["hidden"], s["labels"], LR, BETAS, ADAM_EPS, ignore_index=IGNORE,
                                               reduction=red, threads=16, workspace=s["workspace"])
    return loss, grad_hidden, head.weight, head.master, head.exp_avg, head.exp_avg_sq


def work(case):
    N, H, V = case["N"], case["H"], case["V"]
    size = 4 if case["dtype"] == "fp32" else 2
    inputs = N * H * size + V * H * size + N * 8
    flops = 2 * N * H * V
    if case["kind"] == "forward":
        return {"bytes": inputs + 8 * N, "flops": flops}
    outputs = N * H * size + V * H * size + 4
    if case["kind"] == "head":  # gradients to the host, master and moments read and written, weights back
        outputs += V * H * (2 * size + 24)
    return {"bytes": inputs + outputs, "flops": 3 * flops}


def tolerance(case):
    # The same call in other chunk sizes, each entry's difference over the larger of itself and the
    # result's root mean square in brackets:
    if case["dtype"] == "fp32":  # dW 1.5e-7 [3e-6] at V = 4096; dH sums V terms, and sqrt(V) grows sixfold
        return {"rel": 1e-5, "max": 1e-3}
    if case["kind"] == "forward":  # float32 outputs, 6e-8 from float64: only the order of the sums
        return {"rel": 1e-6, "max": 1e-4}
    # 16-bit gradients round at the stored exponentials, the scaled hidden rows, a running dW and the
    # outputs: dW 1.9e-3 to 4.5e-3 [0.07 to 0.66: rows of frequent ids are far above the root mean
    # square, and their entries are sums of terms that cancel]; dH 1e-4 [8e-3].
    return {"rel": 1e-2, "max": 0.99}


def exact(case, seed):
    hidden, weight, labels, gamma = _inputs(case, seed)
    N, H, V, kind, red = case["N"], case["H"], case["V"], case["kind"], case["reduction"]
    x, w = hidden.double(), weight.double()
    if kind == "rmsnorm":
        h, gam = x, gamma.double()
        r = (h.square().mean(1, keepdim=True) + RMS_EPS).rsqrt()
        x = h * r * gam
    valid = labels != IGNORE
    count = int(valid.sum())
    scale = 1.0 if red != "mean" else (1.0 / count if count else 0.0)
    token, lse = torch.zeros(N, dtype=torch.float64, device=x.device), torch.zeros(N, dtype=torch.float64, device=x.device)
    back = kind != "forward"
    dx, dw = (torch.empty_like(x), torch.zeros_like(w)) if back else (None, None)
    step = max(1, (1 << 28) // V)
    for i in range(0, N, step):
        z = x[i:i + step] @ w.T
        y, ok = labels[i:i + step].clamp(min=0), valid[i:i + step]
        lse[i:i + step] = torch.logsumexp(z, 1)
        token[i:i + step] = torch.where(ok, lse[i:i + step] - z.gather(1, y[:, None])[:, 0], 0.0)
        if back:
            z = torch.exp(z - lse[i:i + step, None])
            z[torch.arange(len(y), device=z.device), y] -= 1.0
            z *= (ok.double() * scale)[:, None]
            dx[i:i + step] = z @ w
            dw += z.T @ x[i:i + step]
        del z
    loss = token.sum() * scale
    if kind == "forward":
        return (token, lse) if red == "none" else loss
    if kind == "rmsnorm":
        dh = r * gam * dx - r ** 3 * h * (h * gam * dx).sum(1, keepdim=True) / H
        return loss, dh, (dx * h * r).sum(0), dw
    if kind == "head":
        m, v = (1 - BETAS[0]) * dw, (1 - BETAS[1]) * dw.square()
        p = w - LR * (m / (1 - BETAS[0])) / ((v / (1 - BETAS[1])).sqrt() + ADAM_EPS)
        return loss, dx, p, p.cpu(), m.cpu(), v.cpu()
    return loss, dx, dw
