"""GPU parity of the fp32 contractions: 128x128 tiles of fp32 values split
into three bf16 terms, with a second pass in fp32 for tiles whose sums are not
finite. Tile edges in every dimension through the fused and the split entry
points against the fp64 oracle; operand magnitudes whose bf16 terms overflow
or vanish; infinite weights that mask vocabulary entries."""
import numpy as np
import pytest
import torch

import kd_inputs as ki
from oracle import kd_topk_kl
from tests.helpers import TOL, oracle_inputs, rel_max, to64

pytestmark = pytest.mark.gpu


def _inputs(N, D, V, K, seed):
    dev = "cuda"
    idx, logit = ki.make_teacher(N, K, V, dev, seed=ki.SEED_TEACHER + seed)
    return dict(hidden=ki.make_hidden(N, D, torch.float32, dev, seed=ki.SEED_HIDDEN + seed),
                W=ki.make_weight(V, D, torch.float32, dev, seed=ki.SEED_W + seed, std=0.05),
                teacher_idx=idx, teacher_logit=logit, ignore=None)


def _args(inp):
    return inp["hidden"], inp["W"], inp["teacher_idx"], inp["teacher_logit"]


def _grads_close(out, ref, tol):
    assert rel_max(to64(out["grad_hidden"]), ref["grad_hidden"]) <= tol
    assert rel_max(to64(out["grad_W"]), ref["grad_W"]) <= tol


@pytest.mark.parametrize("N", [1, 127, 129, 257])
@pytest.mark.parametrize("D,V", [(64, 3), (128, 127), (192, 129), (64, 256), (320, 383),
                                 (64, 1281)])
def test_tile_edges(gpu_lib, N, D, V):
    kd, tol = gpu_lib, TOL["f32"]
    inp = _inputs(N, D, V, min(V, 9), seed=N + V)
    print(f"[f32] N={N} D={D} V={V}", flush=True)
    ref = kd_topk_kl(**oracle_inputs(inp), tau=0.8)
    out = kd.fwd_bwd(*_args(inp), tau=0.8, loss_per_token=True)
    f = kd.fwd(*_args(inp), tau=0.8, loss_per_token=True)
    b = kd.bwd(*_args(inp), f["saved_logz"], tau=0.8)
    torch.cuda.synchronize()
    for o in (out, f):
        assert abs(float(o["loss"]) - ref["loss"]) <= tol["loss"] * abs(ref["loss"])
        assert rel_max(to64(o["loss_per_token"]), ref["loss_per_token"]) <= tol["loss"]
    assert rel_max(to64(f["saved_logz"]), ref["logZ"]) <= tol["loss"]
    _grads_close(out, ref, tol["grad"])
    _grads_close(b, ref, tol["grad"])


@pytest.mark.parametrize("scale", [1e-20, 1e-3, 1e3, 1e28])
def test_operand_magnitudes(gpu_lib, scale):
    """hidden times `scale` and W over it: the logits stay, the operands are
    large or as small as 1e-30 (their last bf16 term then stands at 1e-35,
    still above bf16's smallest normal 1.2e-38). Powers of ten are not exact
    in fp32, so the oracle reads the scaled inputs."""
    kd, tol = gpu_lib, TOL["f32"]
    inp = _inputs(150, 128, 300, 9, seed=3)
    inp["hidden"] = (inp["hidden"].double() * scale).float()
    inp["W"] = (inp["W"].double() / scale).float()
    ref = kd_topk_kl(**oracle_inputs(inp))
    out = kd.fwd_bwd(*_args(inp), loss_per_token=True)
    torch.cuda.synchronize()
    assert abs(float(out["loss"]) - ref["loss"]) <= tol["loss"] * abs(ref["loss"])
    _grads_close(out, ref, tol["grad"])


def test_operand_past_the_largest_bf16(gpu_lib):
    """One hidden feature of 3.4e38, finite in fp32 and infinite once rounded to
    bf16, against weights of 1.2e-38 to 2.4e-38 (logits of 4 to 8): the tiles
    that meet it are formed again in fp32. The feature's own gradients are left
    out: grad_hidden's column is below fp32's normal range, and grad_W's reads
    the hidden rows times a row factor above 1, which overflows fp32."""
    kd, tol = gpu_lib, TOL["f32"]
    inp = _inputs(150, 128, 300, 9, seed=3)
    g = torch.Generator(device="cpu")
    g.manual_seed(ki.SEED_W)
    inp["hidden"][:, 0] = 3.4e38
    inp["W"][:, 0] = (1.2e-38 * (1 + torch.rand(300, generator=g, dtype=torch.float64))).float()
    ref = kd_topk_kl(**oracle_inputs(inp))
    out = kd.fwd_bwd(*_args(inp), loss_per_token=True)
    f = kd.fwd(*_args(inp), loss_per_token=True)
    torch.cuda.synchronize()
    for r in (out, f):
        assert abs(float(r["loss"]) - ref["loss"]) <= tol["loss"] * abs(ref["loss"])
    assert rel_max(to64(out["grad_hidden"])[:, 1:], ref["grad_hidden"][:, 1:]) <= tol["grad"]
    assert rel_max(to64(out["grad_W"])[:, 1:], ref["grad_W"][:, 1:]) <= tol["grad"]


def test_masked_vocabulary_by_infinite_weights(gpu_lib):
    """A constant hidden feature and W = -inf in its column for some vocabulary
    entries: their logits are -inf, their probability is 0, and the loss is the
    one over the other entries. The feature's own grad_hidden column is 0 times
    infinity; every other gradient matches the oracle on the entries kept."""
    kd, tol = gpu_lib, TOL["f32"]
    N, D, V, keep = 140, 64, 300, 260
    inp = _inputs(N, D, V, 9, seed=7)
    idx, logit = ki.make_teacher(N, 9, keep, "cuda", seed=11)
    inp["teacher_idx"], inp["teacher_logit"] = idx, logit
    inp["hidden"][:, 0] = 1.0
    inp["W"][keep:, 0] = float("-inf")
    o = oracle_inputs(inp)
    o["W"] = o["W"][:keep]
    ref = kd_topk_kl(**o)
    out = kd.fwd_bwd(*_args(inp), loss_per_token=True)
    f = kd.fwd(*_args(inp), loss_per_token=True)
    torch.cuda.synchronize()
    for r in (out, f):
        assert abs(float(r["loss"]) - ref["loss"]) <= tol["loss"] * abs(ref["loss"])
    assert rel_max(to64(out["grad_W"])[:keep], ref["grad_W"]) <= tol["grad"]
    assert float(out["grad_W"][keep:].abs().max()) == 0.0
    assert rel_max(to64(out["grad_hidden"])[:, 1:], ref["grad_hidden"][:, 1:]) <= tol["grad"]


def test_nan_input_reaches_the_outputs(gpu_lib):
    """A NaN in one hidden row: that token's loss and gradient row are NaN, the
    other tokens' are finite and unchanged."""
    kd = gpu_lib
    inp = _inputs(200, 64, 300, 9, seed=5)
    clean = kd.fwd_bwd(*_args(inp), loss_per_token=True)
    bad = dict(inp, hidden=inp["hidden"].clone())
    bad["hidden"][17, 5] = float("nan")
    out = kd.fwd_bwd(*_args(bad), loss_per_token=True)
    torch.cuda.synchronize()
    keep = np.arange(200) != 17
    assert np.isnan(to64(out["loss_per_token"])[17])
    assert np.isnan(to64(out["grad_hidden"])[17]).all()
    assert rel_max(to64(out["loss_per_token"])[keep], to64(clean["loss_per_token"])[keep]) <= 1e-6
    assert rel_max(to64(out["grad_hidden"])[keep], to64(clean["grad_hidden"])[keep]) <= 1e-5
