"""Teachers whose entries crowd few vocabulary tiles (K a large part of V): every
256x256 or 128x128 tile then has more entries than threads. Fused and split
entry points against the fp64 oracle."""
import pytest
import torch

import kd_inputs as ki
from oracle import kd_topk_kl
from tests.helpers import TOL, oracle_by_row_blocks, rel_max, to64

pytestmark = pytest.mark.gpu


def _check(kd, N, D, V, K, dtype, masked):
    tol, dev = TOL[dtype], "cuda"
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    h = ki.make_hidden(N, D, tdt, dev, seed=ki.SEED_HIDDEN + 81)
    W = ki.make_weight(V, D, tdt, dev, seed=ki.SEED_W + 81)
    idx, logit = ki.make_teacher(N, K, V, dev, seed=ki.SEED_TEACHER + 81)
    ignore = None
    if masked:
        g = torch.Generator(device="cpu")
        g.manual_seed(ki.SEED_MASK + 81)
        ignore = (torch.rand(N, generator=g) < masked).to(torch.uint8).to(dev)
    print(f"[dense] N={N} D={D} V={V} K={K} {dtype} masked={masked}", flush=True)
    kw = dict(tau=1.2, ignore=ignore)
    out = kd.fwd_bwd(h, W, idx, logit, loss_per_token=True, **kw)
    f = kd.fwd(h, W, idx, logit, loss_per_token=True, **kw)
    b = kd.bwd(h, W, idx, logit, f["saved_logz"], **kw)
    torch.cuda.synchronize()
    ref = oracle_by_row_blocks(kd_topk_kl, to64(h), to64(W), to64(idx), to64(logit), 1.2,
                               ignore=to64(ignore), block=128)
    for r in (out, f):
        assert abs(float(r["loss"]) - ref["loss"]) <= tol["loss"] * abs(ref["loss"])
        assert rel_max(to64(r["loss_per_token"]), ref["loss_per_token"]) <= tol["loss"]
    for r in (out, b):
        assert rel_max(to64(r["grad_hidden"]), ref["grad_hidden"]) <= tol["grad"]
        assert rel_max(to64(r["grad_W"]), ref["grad_W"]) <= tol["grad"]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("N,D,V,K,masked", [
    (190, 128, 351, 351, 0.0),      # the whole vocabulary, small tiles
    (700, 64, 300, 290, 0.4),
    (260, 64, 2000, 1500, 0.9),
    (1100, 64, 9000, 2500, 0.0),    # bf16: 180 tiles of 256, about 18000 entries in each
])
def test_crowded_tiles(gpu_lib, N, D, V, K, masked, dtype):
    _check(gpu_lib, N, D, V, K, dtype, masked)


@pytest.mark.parametrize("N,K,masked", [
    (256, 128, 0.0), (256, 129, 0.0),     # entries of a tile kept in registers, read twice
    (300, 129, 0.3), (254, 129, 0.0),
    (64, 512, 0.0), (64, 513, 0.0), (64, 512, 0.5),
    (1, 4096, 0.0), (9, 4096, 0.0),
])
def test_entries_per_tile(gpu_lib, N, K, masked):
    _check(gpu_lib, N, 64, 5000, K, "bf16", masked)
