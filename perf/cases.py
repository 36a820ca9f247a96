"""Performance cases of the fused chunked top-K KL loss.

Each case is one pass of the loss as a training or evaluation program runs it,
through the package's public calls: the fused forward + backward, the autograd
function in both schedules, the forward alone, the split forward and backward,
and the allocation-free call; bf16 and fp32; with and without ignored tokens;
from a few dozen tokens to the 32K-token benchmark step. Inputs are drawn on
the GPU from the seed: hidden ~ N(0, 1), W ~ N(0, 0.02), K distinct vocabulary
indices per token, teacher logits N(0, 3) sorted descending.
"""
import math

import torch

import paper_2608_03796_amd as kd

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
NOALLOC_CHUNK_BYTES = 160 << 20  # one chunk's gradient rows in the static scratch

# call: fused    kd.fwd_bwd, outputs and workspace kept by the caller
#       autograd topk_kl_loss(...).backward(), schedule "fused"
#       recompute topk_kl_loss(...).backward(), schedule "recompute"
#       split    kd.fwd, then kd.bwd with per-token upstream gradients
#       eval     kd.fwd with per-token losses (no gradients)
#       noalloc  kd.fwd_bwd_noalloc, outputs kept by the caller
BASE = dict(call="fused", dtype="bf16", N=4096, D=4096, V=131072, K=100, chunk=4096, tau=1.0,
            ignored=0.0, logprobs=False, accumulate=False, keep_ws=True)


def _case(name, **kw):
    return dict(BASE, name=name, **kw)


def listed():
    return [
        # the repository's smallest workload: a toy head in fp32, launches and latency
        _case("tiny_fp32", dtype="f32", N=256, D=256, V=4096, K=16, chunk=64),
        # one short training sample through autograd with default arguments
        # (workspace allocated by the call), a tenth of its tokens masked
        _case("short_autograd", call="autograd", N=77, D=768, V=32003, K=20, ignored=0.1,
              keep_ws=False),
        # a 512-token step of a small model in a captured or allocation-free loop
        _case("noalloc_512", call="noalloc", N=512, D=1024, V=32000, K=64, chunk=256),
        # one micro-batch of gradient accumulation into fp32 grad_W with cached
        # log-probabilities (partial-mass teacher), ragged N and V
        _case("micro2k_accumulate", N=2000, D=2048, V=50021, K=50, chunk=1024, logprobs=True,
              accumulate=True),
        # a small model trained in fp32
        _case("f32_2k", dtype="f32", N=2048, D=1024, V=32000, K=50, chunk=1024, tau=2.0),
        # fp32, the split entry points with per-token loss weights, ragged sizes and chunk
        _case("f32_split_ragged", call="split", dtype="f32", N=1000, D=768, V=30011, K=32,
              chunk=300, ignored=0.2),
        # one 4K-token sequence at the benchmark's head size
        _case("loss4k"),
        # evaluation: losses of 8K tokens, no gradients
        _case("eval8k", call="eval", N=8192),
        # the memory-saving autograd schedule on instruction data: a third of the
        # tokens are prompt and masked; odd sizes
        _case("recompute_ragged", call="recompute", N=6001, D=2560, V=100003, chunk=1500,
              ignored=0.35),
        # the packed-documents training step through autograd
        _case("packed_autograd", call="autograd", N=32768, D=3072, V=128256, chunk=2048, tau=2.0,
              ignored=0.05),
        # the headline benchmark step
        _case("loss32k", N=32768),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: N 64..32768, D 256..4096, V 4096..131072,
    K 1..128, any chunk, at no more than the largest listed case's cost."""
    while True:
        c = dict(BASE)
        c["call"] = rng.choice(["fused", "fused", "autograd", "recompute", "split", "eval",
                                "noalloc"])
        c["dtype"] = rng.choice(["bf16", "bf16", "bf16", "f32"])
        c["N"] = _log_int(rng, 64, 32768)
        c["D"] = 64 * _log_int(rng, 4, 64)
        c["V"] = _log_int(rng, 4096, 131072)
        c["K"] = _log_int(rng, 1, 128)
        c["chunk"] = rng.choice([_log_int(rng, 64, 4096), 256 * rng.randint(1, 16)])
        c["tau"] = rng.choice([0.5, 1.0, 1.0, 2.0])
        c["ignored"] = rng.choice([0.0, 0.0, 0.05, round(rng.uniform(0.0, 0.9), 2)])
        c["logprobs"] = rng.random() < 0.25
        c["accumulate"] = c["call"] in ("fused", "noalloc") and rng.random() < 0.3
        c["keep_ws"] = rng.random() < 0.7
        eb = 2 if c["dtype"] == "bf16" else 4
        if c["call"] == "noalloc" and c["chunk"] * c["V"] * eb > NOALLOC_CHUNK_BYTES:
            continue
        ndv = c["N"] * c["D"] * c["V"]
        if ndv <= (32768 * 4096 * 131072 if eb == 2 else 32768 * 4096 * 4096) // 2:
            return c


def _distinct(N, K, V, g, dev):
    """K distinct indices per row: sorted draws from [0, V - K] plus 0..K-1."""
    x = torch.randint(0, V - K + 1, (N, K), generator=g, device=dev).sort(dim=1).values
    x = x + torch.arange(K, device=dev)
    order = torch.rand(N, K, generator=g, device=dev).argsort(dim=1)
    return x.gather(1, order).to(torch.int32).contiguous()


def _randn(n, d, std, dtype, g, dev):
    x = torch.empty(n, d, dtype=dtype, device=dev)
    for s in range(0, n, 32768):
        e = min(n, s + 32768)
        x[s:e] = torch.randn(e - s, d, generator=g, device=dev) * std
    return x


def _inputs(case, seed):
    dev = torch.device("cuda", torch.cuda.current_device())
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    N, D, V, K = case["N"], case["D"], case["V"], case["K"]
    dt = DTYPES[case["dtype"]]
    s = {"hidden": _randn(N, D, 1.0, dt, g, dev), "W": _randn(V, D, 0.02, dt, g, dev)}
    s["teacher_idx"] = _distinct(N, K, V, g, dev)
    logit = (torch.randn(N, K, generator=g, device=dev) * 3).sort(dim=1, descending=True).values
    if case["logprobs"]:
        # log-probabilities over the whole vocabulary: a retained mass of 0.7 to 1
        mass = 0.7 + 0.3 * torch.rand(N, 1, generator=g, device=dev)
        logit = torch.log_softmax(logit, dim=1) + mass.log()
    s["teacher_logit"] = logit.contiguous()
    s["ignore"] = None
    if case["ignored"] > 0:
        s["ignore"] = (torch.rand(N, generator=g, device=dev) < case["ignored"]).to(torch.uint8)
        s["ignore"][0] = 0
    s["grad_W0"] = None
    if case["accumulate"]:
        # the gradient sum of earlier micro-batches
        s["grad_W0"] = _randn(V, D, 1e-5, torch.float32, g, dev)
    s["token_grad"] = None
    if case["call"] == "split":
        s["token_grad"] = torch.rand(N, generator=g, device=dev) * (2.0 / N)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    dev = s["hidden"].device
    N, D, V = case["N"], case["D"], case["V"]
    code = kd.KD_BF16 if case["dtype"] == "bf16" else kd.KD_F32
    s["call"] = case["call"]
    s["accumulate"] = case["accumulate"]
    s["kw"] = dict(tau=case["tau"], ignore=s["ignore"], chunk=case["chunk"],
                   teacher_logprobs=case["logprobs"])
    s["ws"] = None
    if case["keep_ws"] and case["call"] != "noalloc":
        s["ws"] = kd.alloc_workspace(N, D, V, case["K"], case["chunk"], case["tau"], code, dev)
    if case["call"] in ("fused", "noalloc"):
        s["out"] = {"loss": torch.empty((), dtype=torch.float32, device=dev),
                    "loss_per_token": torch.empty(N, dtype=torch.float32, device=dev),
                    "grad_hidden": torch.empty(N, D, dtype=s["hidden"].dtype, device=dev),
                    "grad_W": s["grad_W0"] if case["accumulate"] else torch.empty(
                        V, D, dtype=torch.float32, device=dev)}
    if case["call"] in ("autograd", "recompute"):
        s["hidden"].requires_grad_(True)
        s["W"].requires_grad_(True)
    return s


def run(s):
    t = (s["hidden"], s["W"], s["teacher_idx"], s["teacher_logit"])
    call, kw = s["call"], s["kw"]
    if call == "fused":
        return kd.fwd_bwd(*t, workspace=s["ws"], out=s["out"], loss_per_token=True,
                          accumulate_grad_W=s["accumulate"], **kw)
    if call == "noalloc":
        return kd.fwd_bwd_noalloc(*t, out=s["out"], loss_per_token=True,
                                  accumulate_grad_W=s["accumulate"], **kw)
    if call == "eval":
        return kd.fwd(*t, loss_per_token=True, workspace=s["ws"], **kw)
    if call == "split":
        f = kd.fwd(*t, loss_per_token=True, workspace=s["ws"], **kw)
        b = kd.bwd(*t, f["saved_logz"], grad_loss_per_token=s["token_grad"], workspace=s["ws"],
                   **kw)
        return {**f, **b}
    s["hidden"].grad = None
    s["W"].grad = None
    schedule = "fused" if call == "autograd" else "recompute"
    loss = kd.topk_kl_loss(*t, schedule=schedule, workspace=s["ws"], **kw)
    loss.backward()
    return {"loss": loss.detach(), "grad_hidden": s["hidden"].grad, "grad_W": s["W"].grad}


def _valid(case):
    return case["N"] * (1.0 - case["ignored"])


def work(case):
    N, D, V, K = case["N"], case["D"], case["V"], case["K"]
    eb = 2 if case["dtype"] == "bf16" else 4
    nv = _valid(case)
    # inputs: the tokens that are not ignored, W, the teacher arrays, the mask
    b = nv * D * eb + V * D * eb + nv * K * 8 + (N if case["ignored"] > 0 else 0)
    contractions = {"eval": 1, "split": 4, "recompute": 4}.get(case["call"], 3)
    if case["call"] != "eval":
        gw = eb if case["call"] in ("autograd", "recompute") else 4
        b += N * D * eb + V * D * gw * (2 if case["accumulate"] else 1)
    if case["call"] in ("split", "recompute"):
        b += nv * D * eb + V * D * eb  # a second call reads its inputs again
    return {"bytes": float(b), "flops": 2.0 * contractions * nv * D * V}


def tolerance(case):
    # bf16: the gradient of the logits and grad_hidden are rounded to 8 bits of
    # mantissa (2^-9 each): about 2.5e-3 against exact; fp32: sums of up to V terms
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-5}


def exact(case, seed):
    """The dense loss and its gradients in float64, a block of tokens at a time."""
    s = _inputs(case, seed)
    N, V, tau = case["N"], case["V"], case["tau"]
    dev = s["hidden"].device
    W = s["W"].double()
    valid = torch.ones(N, dtype=torch.bool, device=dev)
    if s["ignore"] is not None:
        valid = s["ignore"] == 0
    n_valid = int(valid.sum())
    grads = case["call"] != "eval"
    lpt = torch.zeros(N, dtype=torch.float64, device=dev)
    logz = torch.zeros(N, dtype=torch.float64, device=dev)
    gh = torch.zeros(N, case["D"], dtype=torch.float64, device=dev) if grads else None
    gw = torch.zeros(V, case["D"], dtype=torch.float64, device=dev) if grads else None
    rows = valid.nonzero().squeeze(1)
    for r in rows.split(2048):
        h = s["hidden"][r].double()
        idx = s["teacher_idx"][r].long()
        u = s["teacher_logit"][r].double()
        logp = u if case["logprobs"] else torch.log_softmax(u / tau, dim=1)
        p = logp.exp()
        mass = p.sum(dim=1)
        y = (h @ W.t()) / tau
        lz = torch.logsumexp(y, dim=1)
        logz[r] = lz
        lpt[r] = (p * logp).sum(1) - (p * y.gather(1, idx)).sum(1) + mass * lz
        if grads:
            g = torch.full_like(lz, 1.0 / n_valid)
            if s["token_grad"] is not None:
                g = s["token_grad"][r].double()
            G = y.sub_(lz[:, None]).exp_().mul_(mass[:, None])
            G.scatter_add_(1, idx, -p)
            G.mul_((g / tau)[:, None])
            gh[r] = G @ W
            gw += G.t() @ h
    out = {"loss": lpt.sum() / n_valid}
    if case["call"] in ("fused", "noalloc", "eval", "split"):
        out["loss_per_token"] = lpt
    if case["call"] in ("eval", "split"):
        out["saved_logz"] = logz
    if grads:
        out["grad_hidden"] = gh
        out["grad_W"] = gw if s["grad_W0"] is None else gw + s["grad_W0"].double()
    return out
