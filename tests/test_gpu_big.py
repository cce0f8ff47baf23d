"""The large tile kernel of 3- and 4-bit codes against the CPU oracle where its blocks, steps and sets end, and the device's lookup of
a step's pairs with as many experts as there can be."""
import numpy as np
import pytest
import torch

import workload as W
from oracle import moe_oracle as O
from paper_2312_17238_amd import binding as B

from harness import Model, run_teacher_forced
from test_gpu_tile import one_step, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt,sg", [((4, 64), 0), ((4, 64), 2), ((4, 128), 0), ((3, 64), 0), ((3, 64), 1)])
@pytest.mark.parametrize("H,F,Bn", [(128, 256, 127), (384, 128, 128), (256, 640, 129), (640, 384, 257)])
def test_ends_of_blocks_and_sets(fmt, sg, H, F, Bn):
    """One expert's tokens one short of a block of 128, a block, one more and two blocks and one; contractions of two to ten units, whose last set
    holds two or all of its four (bounds on y: harness.check_y)."""
    model = Model(1, H, F, 1, 1, [fmt], 1, 0, 1e-5, max_batch=Bn, seed=81, scale_group=sg)
    B.moe_ctx_set_option(model.stack.ctx, "mfma_form", 6)
    B.moe_ctx_set_option(model.stack.ctx, "tile_tokens", 192)
    run_teacher_forced(model, W.hidden_ar1(81, 1, Bn, H), O.expert_ffn, rows=lambda t, l: sorted({0, 31, 32, 95, 96, Bn - 2, Bn - 1}))
    model.close()


@pytest.mark.parametrize("fmt,sg", [((4, 64), 0), ((3, 64), 0)])
@pytest.mark.parametrize("H,F,Bn", [(64, 192, 40), (192, 320, 70), (448, 64, 100)])
def test_rows_of_an_odd_number_of_units(fmt, sg, H, F, Bn):
    """The second unit of a row's last step does not exist; several experts, blocks of one to four tiles."""
    run(fmt, sg, H, F, 3, 2, 3, Bn, tile=192)


@pytest.mark.parametrize("K,Bn", [(4, 16), (4, 17), (3, 64), (4, 64)])
@pytest.mark.parametrize("form", [5, 6])
def test_pairs_found_on_the_device_among_16_experts(K, Bn, form):
    """64, 68, 192 and 256 pairs: a queued step, whose kernels look them up, gives the bits of one that waits (form 5: the host's tables)."""
    model = Model(1, 128, 256, 16, K, [(4, 64)], 16, 0, 1e-5, max_batch=Bn, seed=82)
    x = W.hidden_ar1(82, 1, Bn, 128)[0].to(model.stack.device)
    bits = one_step(model, x, form)
    for _ in range(2):                                   # the first step fills the slots and waits as well
        out = torch.empty_like(x)
        model.stack.step_layer(0, x, out)
        model.stack.synchronize()
    assert model.stack.total_stats()["steps_device_routed"] > 0
    assert (model.stack.read_y(Bn, 128).view(np.uint32) == bits).all()
    model.close()
