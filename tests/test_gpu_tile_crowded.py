"""Tile kernels, tokens that crowd to a few experts: w2's contraction takes other parts than with an even routing, the same ones
whether the host saw the routing and whatever the cache held.  Against the CPU oracle."""
import numpy as np
import pytest
import torch

import workload as W
from oracle import moe_oracle as O
from paper_2312_17238_amd import binding as B

from harness import Model, check_y, oracle_routing, oracle_y, say

pytestmark = pytest.mark.gpu

# (format, scale group, H, F, E, K, tokens, tokens per block): every size of block, one and two of an expert, pairs found by ballots and
# sorted; contractions whose last part is short; half of the even routing's blocks and fewer
CASES = [((3, 64), 0, 4096, 1088, 8, 2, 12, 0), ((2, 16), 0, 4096, 1088, 8, 2, 12, 0), ((2, 16), 16, 2048, 1344, 8, 2, 40, 32), ((4, 64), 0, 4096, 1088, 8, 2, 64, 32),
         ((4, 32), 0, 2048, 1344, 13, 3, 20, 0), ((3, 64), 4, 4096, 2112, 8, 2, 150, 192), ((4, 128), 0, 4096, 2176, 8, 1, 300, 192), ((4, 64), 16, 1856, 1344, 6, 2, 16, 0)]


def crowd(kind, Bn, H):
    x = W.hidden_ar1(76, 1, Bn, H)[0]
    return x[:1].expand(Bn, H).contiguous() if kind == "one" else x[torch.arange(Bn) % 3].contiguous() if kind == "three" else x


@pytest.mark.parametrize("fmt,sg,H,F,E,K,Bn,tile", CASES)
def test_crowded_tokens(fmt, sg, H, F, E, K, Bn, tile):
    ys, first = {}, {}
    for k in (E, K + 1):
        model = Model(1, H, F, E, K, [fmt], k, 0, 1e-5, max_batch=Bn, seed=77, scale_group=sg, init_policy=1)
        B.moe_ctx_set_option(model.stack.ctx, "mfma_form", 6)
        B.moe_ctx_set_option(model.stack.ctx, "tile_tokens", tile)
        for kind in ("one", "three", "spread"):
            x = crowd(kind, Bn, H).to(model.stack.device)
            out, got = torch.empty_like(x), []
            for routed in (1, 0):
                B.moe_ctx_set_option(model.stack.ctx, "device_routing", routed)
                torch.cuda.synchronize()
                model.stack.step_layer(0, x, out)
                got.append(model.stack.read_y(Bn, H).copy().view(np.uint32))
            assert (got[0] == got[1]).all()
            assert (ys.setdefault(kind, got[0]) == got[0]).all()
            if k == E:
                routing = oracle_routing(model, 0, x.cpu().numpy())
                rel = [check_y(got[0].view(np.float32)[b], oracle_y(model, 0, routing[b][0], routing[b][1], routing[b][2], O.expert_ffn), f"{kind} b={b}")[1]
                       for b in sorted({0, Bn // 2, Bn - 1})]
                say(f"crowded {fmt} {sg} {H}x{F} E={E} K={K} B={Bn} {kind}: rel {max(rel):.2e}")
        model.close()
    # the first token is the same in all three; its sums are not added in the same order
    assert (ys["one"][0] != ys["spread"][0]).any()


# The same (format, .., tokens per block), where the even routing's plan has several parts and all tokens at the same experts leave one; what the plan
# says of them is seen by test_plans.py.  Tiles of 16 and 32, both large kernels of 2-bit codes and the one of the others (their 600 pairs sorted).
ONE_PART = [((4, 32), 0, 4352, 512, 8, 1, 100, 0), ((4, 32), 8, 4352, 512, 16, 1, 128, 0), ((4, 64), 0, 4352, 512, 16, 2, 100, 0), ((4, 128), 2, 4352, 512, 16, 1, 128, 0),
            ((3, 64), 4, 4352, 512, 16, 1, 128, 0), ((2, 16), 0, 4352, 512, 16, 1, 128, 0), ((2, 16), 16, 4352, 512, 8, 1, 100, 0), ((2, 16), 0, 4352, 512, 16, 2, 100, 32),
            ((2, 16), 0, 5632, 512, 13, 3, 200, 192), ((2, 16), 16, 5632, 512, 13, 3, 200, 0), ((3, 64), 0, 5632, 512, 13, 3, 200, 192), ((4, 64), 16, 5632, 512, 13, 3, 200, 192)]


@pytest.mark.parametrize("fmt,sg,H,F,E,K,Bn,tile", ONE_PART)
def test_several_parts_become_one(fmt, sg, H, F, E, K, Bn, tile):
    """Behind a step of other tokens, whose rows the crowded one must not read."""
    model = Model(1, H, F, E, K, [fmt], E, 0, 1e-5, max_batch=Bn, seed=78, scale_group=sg)
    B.moe_ctx_set_option(model.stack.ctx, "mfma_form", 6)
    B.moe_ctx_set_option(model.stack.ctx, "tile_tokens", tile)
    for routed in (1, 0):
        B.moe_ctx_set_option(model.stack.ctx, "device_routing", routed)
        for kind in ("spread", "one"):
            x = crowd(kind, Bn, H).to(model.stack.device)
            out = torch.empty_like(x)
            torch.cuda.synchronize()
            model.stack.step_layer(0, x, out)
            y = model.stack.read_y(Bn, H).copy()
        routing = oracle_routing(model, 0, x[:1].cpu().numpy())[0]
        ref = oracle_y(model, 0, routing[0], routing[1], routing[2], O.expert_ffn)
        for b in (0, Bn // 2, Bn - 1):
            check_y(y[b], ref, f"routed={routed} b={b}")
        assert (y.view(np.uint32) == y[:1].view(np.uint32)).all()        # equal tokens
    model.close()
