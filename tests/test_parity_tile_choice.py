"""bf16 contractions in 256x256 and in 128x128 tiles: problems on both sides of
each contraction's rule, with ragged tiles of both sizes and split last
rounds, through the fused and the split entry points, against the fp64
oracle."""
import pytest
import torch

import kd_inputs as ki
from oracle import kd_topk_kl
from tests.helpers import TOL, oracle_by_row_blocks, rel_max, to64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,D,V,masked,tau", [
    (256, 128, 32768, 0.0, 1.3),     # 128 projection tiles: small ones
    (256, 128, 32769, 0.0, 1.3),     # 129: large ones; one column in the last
    (257, 64, 33100, 0.3, 1.3),      # large, a last token tile of one row
    (259, 1344, 33000, 0.0, 1.3),    # all three contractions large, ragged each way
    (259, 1344, 33000, 0.4, 1.3),
    (128, 192, 33100, 0.0, 1.3),     # dW: two K steps in small tiles
    (129, 192, 33100, 0.0, 1.3),     # dW: three K steps in large ones
    (300, 2048, 700, 0.0, 1.3),      # dH: 16 tiles
    (200, 2048, 700, 0.0, 1.3),      # dH: 8 tiles
    (1000, 64, 600, 0.1, 1.3),       # dW: few tiles, split along the tokens
    (1, 64, 5, 0.0, 1.3),
    (512, 64, 33000, 0.0, 1.3),    # 258 projection tiles: 256 large, the last two as small ones
    (512, 64, 33000, 0.4, 1.3),
    (512, 64, 33000, 0.1, 0.02),   # rows that fall back to a tile's own max in both tile sizes
])
def test_tile_choice(gpu_lib, N, D, V, masked, tau):
    kd, tol, dev, K = gpu_lib, TOL["bf16"], "cuda", min(V, 11)
    h = ki.make_hidden(N, D, torch.bfloat16, dev, seed=ki.SEED_HIDDEN + 71)
    W = ki.make_weight(V, D, torch.bfloat16, dev, seed=ki.SEED_W + 71)
    idx, logit = ki.make_teacher(N, K, V, dev, seed=ki.SEED_TEACHER + 71)
    ignore = None
    if masked:
        g = torch.Generator(device="cpu")
        g.manual_seed(ki.SEED_MASK + 71)
        ignore = (torch.rand(N, generator=g) < masked).to(torch.uint8).to(dev)
    print(f"[tiles] N={N} D={D} V={V} masked={masked} tau={tau}", flush=True)
    ref = oracle_by_row_blocks(kd_topk_kl, to64(h), to64(W), to64(idx), to64(logit), tau,
                               ignore=to64(ignore), block=128)
    kw = dict(tau=tau, ignore=ignore)
    ws = torch.full((kd.workspace_size(N, D, V, K, 4096, tau),), 0xff, dtype=torch.uint8,
                    device=dev)
    out = kd.fwd_bwd(h, W, idx, logit, loss_per_token=True, workspace=ws, **kw)
    ws.fill_(0xff)
    f = kd.fwd(h, W, idx, logit, loss_per_token=True, workspace=ws, **kw)
    ws.fill_(0xff)
    b = kd.bwd(h, W, idx, logit, f["saved_logz"], workspace=ws, **kw)
    gw = out["grad_W"].clone()
    kd.fwd_bwd(h, W, idx, logit, grad_W_out=gw, accumulate_grad_W=True, workspace=ws, **kw)
    torch.cuda.synchronize()
    for r in (out, f):
        assert abs(float(r["loss"]) - ref["loss"]) <= tol["loss"] * abs(ref["loss"])
        assert rel_max(to64(r["loss_per_token"]), ref["loss_per_token"]) <= tol["loss"]
    for r in (out, b):
        assert rel_max(to64(r["grad_hidden"]), ref["grad_hidden"]) <= tol["grad"]
        assert rel_max(to64(r["grad_W"]), ref["grad_W"]) <= tol["grad"]
    # the same sum twice, each rounded to fp32
    assert rel_max(to64(gw), 2 * to64(out["grad_W"])) <= 1e-6
