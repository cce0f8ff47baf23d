"""Steps of more than 256 pairs, whose pairs one block sorts by expert, at the ends of its chunks of 64 pairs, and the last kernel of a
step with few and many partial rows of a pair: y against the CPU oracle, and the experts a queued step is booked with."""
import numpy as np
import pytest
import torch

import workload as W
from oracle import moe_oracle as O
from paper_2312_17238_amd import binding as B

from harness import Model, run_teacher_forced
from test_gpu_tile import one_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,K,Bn", [(16, 1, 257), (16, 3, 171), (13, 4, 256), (1, 1, 320), (16, 4, 1023), (16, 4, 1024), (8, 2, 1024)])
def test_pairs_sorted_by_expert(E, K, Bn):
    """257 to 4096 pairs; a queued step gives the bits of one that waits, and books the same experts (bounds on y: harness.check_y)."""
    model = Model(1, 64, 128, E, K, [(4, 64)], E, 0, 1e-5, max_batch=Bn, seed=91)
    xs = W.hidden_ar1(91, 1, Bn, 64)
    B.moe_ctx_set_option(model.stack.ctx, "mfma_form", 6)
    _, sim, _ = run_teacher_forced(model, xs, O.expert_ffn, rows=lambda t, l: sorted({0, 63, 64, Bn // 2, Bn - 1}))
    x = xs[0].to(model.stack.device)
    bits, out = one_step(model, x, 6), torch.empty_like(x)
    before = model.stack.total_stats()
    model.stack.step_layer(0, x, out)
    model.stack.synchronize()
    after = model.stack.total_stats()
    assert after["steps_device_routed"] == before["steps_device_routed"] + 1
    assert 2 * (after["needed"] - before["needed"]) == before["needed"]          # the two steps before it needed the same ones
    assert (model.stack.read_y(Bn, 64).view(np.uint32) == bits).all()
    model.close()


@pytest.mark.parametrize("K,F,Bn,form", [(1, 256, 3, 6), (3, 2048, 3, 6), (4, 4096, 17, 6), (4, 1024, 16, 5), (2, 4096, 4, 5), (2, 2048, 2, 5)])
def test_rows_added_by_the_last_kernel(K, F, Bn, form):
    """One to four experts a token, w2's contraction whole and in up to eight parts (bounds on y: harness.check_y)."""
    model = Model(1, 128, F, 5, K, [(4, 64)], 5, 0, 1e-5, max_batch=Bn, seed=92)
    B.moe_ctx_set_option(model.stack.ctx, "mfma_form", form)
    B.moe_ctx_set_option(model.stack.ctx, "mfma_min_batch", 1)
    run_teacher_forced(model, W.hidden_ar1(92, 1, Bn, 128), O.expert_ffn)
    model.close()
