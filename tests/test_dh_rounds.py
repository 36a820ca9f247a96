"""dH's last round of tiles split along the vocabulary: row counts on both
sides of a round, with and without ignored tokens (the split is then chosen
on the device), through the fused and the split entry points, against the fp64
oracle."""
import pytest
import torch

import kd_inputs as ki
from oracle import kd_topk_kl
from tests.helpers import TOL, oracle_by_row_blocks, rel_max, to64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("N,D,V,masked", [
    (130, 320, 9000, None),      # few tiles, many ranges
    (600, 4160, 700, None),      # a last tile column of 64 features, few K steps (no split)
    (2100, 8192, 1100, None),    # a whole round and a split rest (bf16: 288 tiles)
    (2100, 8192, 1100, 0.5),     # the device finds fewer tiles than the host
    (2100, 8192, 1100, 0.999),   # a few rows of one tile
    (900, 256, 9000, 0.7),
    (300, 64, 5000, 1.0),        # no rows at all
])
def test_split_last_round(gpu_lib, dtype, N, D, V, masked):
    kd, tol, dev = gpu_lib, TOL[dtype], "cuda"
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    h = ki.make_hidden(N, D, tdt, dev, seed=ki.SEED_HIDDEN + 51, std=min(1.0, (2048 / D) ** 0.5))
    W = ki.make_weight(V, D, tdt, dev, seed=ki.SEED_W + 51)
    idx, logit = ki.make_teacher(N, 9, V, dev, seed=ki.SEED_TEACHER + 51)
    ignore = None
    if masked is not None:
        g = torch.Generator(device="cpu")
        g.manual_seed(ki.SEED_MASK + 51)
        ignore = (torch.rand(N, generator=g) < masked).to(torch.uint8).to(dev)
    print(f"[dh] N={N} D={D} V={V} masked={masked} {dtype}", flush=True)
    ref = oracle_by_row_blocks(kd_topk_kl, to64(h), to64(W), to64(idx), to64(logit), 1.0,
                               ignore=to64(ignore), block=256)
    gh = torch.full((N, D), float("nan"), dtype=tdt, device=dev)
    out = kd.fwd_bwd(h, W, idx, logit, ignore=ignore, out={"grad_hidden": gh}, grad_W=False)
    f = kd.fwd(h, W, idx, logit, ignore=ignore)
    b = kd.bwd(h, W, idx, logit, f["saved_logz"], ignore=ignore, grad_W=False,
               grad_hidden_f32=True)
    torch.cuda.synchronize()
    for r in (out, b):
        assert rel_max(to64(r["grad_hidden"]), ref["grad_hidden"]) <= tol["grad"]
    # two calls give the same bits
    again = kd.fwd_bwd(h, W, idx, logit, ignore=ignore, grad_W=False)
    torch.cuda.synchronize()
    assert torch.equal(again["grad_hidden"], out["grad_hidden"])
