"""The tile kernels' own rounding against 64 bits, on tokens with and without a mean."""
import numpy as np
import pytest
import torch

from paper_2312_17238_amd import binding as B

from harness import Model, oracle_routing, say
from test_gpu_tile import one_step, weights64

pytestmark = pytest.mark.gpu


def errors(fmt, sg, mean, deviation):
    """Relative errors of y against 64 bits (the activations between the halves rounded to fp16 there too), GEMV and tile kernels."""
    H, F = 4096, 4096
    model = Model(1, H, F, 1, 1, [fmt], 1, 0, 1e-5, max_batch=32, seed=67, scale_group=sg)
    x = (mean + deviation * torch.randn(32, H, generator=torch.Generator().manual_seed(67))).to(torch.float16)
    h = np.stack([r[0] for r in oracle_routing(model, 0, x.numpy())]).astype(np.float64)
    w1, w3, w2 = (weights64(m, fmt[1], sg) for m in model.expert_np(0, 0))
    u = h @ w1.T
    y = (u / (1.0 + np.exp(-u)) * (h @ w3.T)).astype(np.float16).astype(np.float64) @ w2.T
    xd = x.to(model.stack.device)
    err = {}
    for name, n, low, tile in (("gemv", 16, 1000, 0), ("16", 16, 1, 16), ("32", 32, 1, 32), ("large", 32, 1, 192)):
        B.moe_ctx_set_option(model.stack.ctx, "mfma_min_batch", low)
        B.moe_ctx_set_option(model.stack.ctx, "tile_tokens", tile)
        g = one_step(model, xd[:n].contiguous(), 5 if name == "gemv" else 6).view(np.float32)
        err[name] = np.linalg.norm(g - y[:n]) / np.linalg.norm(y[:n])
    model.close()
    say(f"tile {fmt} {sg} mean {mean}: {err}")
    return err


@pytest.mark.parametrize("fmt,sg", [((4, 64), 0), ((4, 64), 128), ((4, 128), 0), ((4, 32), 128), ((3, 64), 0), ((3, 64), 128)])
@pytest.mark.parametrize("mean,deviation", [(0.0, 1.0), (0.1, 1.0), (1.0, 0.125)])
def test_error_does_not_grow_with_the_tokens_mean(fmt, sg, mean, deviation):
    """y against 64 bits (the activations between the halves rounded to fp16 there too) beside the GEMV kernels' on the same tokens.
    Those multiply codes with biases of 64 and 1024; the tile kernels' codes have none, so their sums are at least 64 / 8 times
    smaller and so is what rounding them to fp32 leaves.  An a that falls to the other of two fp16 numbers adds an error
    that goes with the square root of it: 1 / sqrt(8), 0.36 of the GEMV kernels' error."""
    err = errors(fmt, sg, mean, deviation)
    assert max(err["16"], err["32"], err["large"]) <= 0.36 * err["gemv"]


@pytest.mark.parametrize("sg", [0, 128])
@pytest.mark.parametrize("mean,deviation", [(0.0, 1.0), (0.1, 1.0), (1.0, 0.125)])
def test_2bit_tiles_no_less_exact_than_the_gemv_kernels(sg, mean, deviation):
    """Steps of two and three tokens of an expert take tiles of 16 where smaller ones take the GEMV kernels, whose zero-point term
    is in fp32: a step's error does not grow with its tokens."""
    err = errors((2, 16), sg, mean, deviation)
    assert err["16"] <= err["gemv"]
