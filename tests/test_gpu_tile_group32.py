"""The tile kernels for 4-bit codes in groups of 32 (two groups a unit, tiles of 16 and 32 tokens only) against the CPU oracle."""
import numpy as np
import pytest

import workload as W
from paper_2312_17238_amd import binding as B

from harness import Model, oracle_routing, say
from test_gpu_tile import one_step, run, weights64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sg", [0, 2, 256])
@pytest.mark.parametrize("H,F,Bn", [(128, 128, 3), (384, 640, 33), (320, 896, 70)])
def test_edges(sg, H, F, Bn):
    """Rows and units that fill no block, no set; several token blocks; runs of one unit and of a row."""
    run((4, 32), sg, H, F, 4, 2, 4, Bn)


@pytest.mark.parametrize("sg,Bn", [(s, b) for s in (0, 16) for b in (1, 15, 16, 17, 32, 33, 100)])
def test_pipelines_in_their_steady_state(sg, Bn):
    """Contractions of several sets, the last one short, every part of w2's several; one expert has every token."""
    run((4, 32), sg, 1344, 6208, 1, 1, 1, Bn, rows={0, Bn // 2, Bn - 1})


def test_offloaded():
    """Fewer slots than needed experts."""
    run((4, 32), 128, 256, 640, 8, 2, 3, 48, T=3, m=2)


@pytest.mark.parametrize("H,F,sg", [(64, 640, 0), (640, 64, 0), (256, 640, 1)])
def test_layers_left_on_the_gemv_kernels(H, F, sg):
    """Rows of a single unit, metadata runs of half a unit."""
    model = Model(1, H, F, 4, 2, [(4, 32)], 4, 0, 1e-5, max_batch=20, seed=73, scale_group=sg)
    x = W.hidden_ar1(73, 1, 20, H)[0].to(model.stack.device)
    assert (one_step(model, x, 6) == one_step(model, x, 5)).all()
    model.close()


@pytest.mark.parametrize("sg", [0, 16])
@pytest.mark.parametrize("Bn", [16, 40])
def test_as_exact_as_the_gemv_kernels(sg, Bn):
    """Error against 64 bits (the activations between the halves rounded to fp16 there too) beside the GEMV kernels' on the same
    tokens: the products' sums are half as long as with groups of 64, the scaling the same, so well below it."""
    H, F = 1024, 2048
    model = Model(1, H, F, 1, 1, [(4, 32)], 1, 0, 1e-5, max_batch=Bn, seed=66, scale_group=sg)
    xs = W.hidden_ar1(66, 1, Bn, H)[0]
    h = np.stack([r[0] for r in oracle_routing(model, 0, xs.numpy())]).astype(np.float64)
    w1, w3, w2 = (weights64(m, 32, sg) for m in model.expert_np(0, 0))
    u = h @ w1.T
    y = (u / (1.0 + np.exp(-u)) * (h @ w3.T)).astype(np.float16).astype(np.float64) @ w2.T
    x = xs.to(model.stack.device)
    tile = one_step(model, x, 6)
    B.moe_ctx_set_option(model.stack.ctx, "mfma_min_batch", 1000)
    gemv = one_step(model, x, 5)
    model.close()
    err = [np.linalg.norm(v.view(np.float32) - y) / np.linalg.norm(y) for v in (tile, gemv)]
    say(f"tile group 32 {sg} B={Bn}: {err[0]:.3g} against {err[1]:.3g}")
    assert err[0] <= 0.8 * err[1]
