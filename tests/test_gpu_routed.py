"""Steps of several tokens through layers whose experts are all on the device: queued without the host seeing the routing, the
kernels find it in device memory.  Same bits as the waiting step's, same counters, the oracle's outputs."""
import numpy as np
import pytest
import torch

import workload as W
from oracle import moe_oracle as O
from paper_2312_17238_amd import binding as B

from harness import Model, check_y, oracle_routing, oracle_y, say

pytestmark = pytest.mark.gpu

# (format, scale group, H, F, E, K, tokens): GEMV kernels with entries of two and of four tokens; 16-token kernels with tiles of 16 and 32, up
# to 256 pairs; tile kernels of each size, with the pairs found by ballots (one chunk of 64 pairs and more, up to 256) and sorted
# (more); an odd number of experts, sixteen of them, three choices; a layer where all are needed.
CASES = [((4, 64), 0, 256, 512, 8, 2, 2), ((3, 64), 0, 256, 512, 16, 3, 5), ((2, 16), 8, 256, 512, 8, 2, 12), ((4, 32), 0, 320, 640, 13, 2, 32),
         ((4, 64), 0, 256, 512, 8, 2, 3), ((4, 64), 4, 512, 640, 13, 3, 21), ((4, 64), 0, 256, 512, 8, 2, 64), ((4, 64), 0, 256, 512, 8, 2, 128),
         ((3, 64), 0, 512, 640, 6, 2, 32), ((3, 64), 2, 512, 640, 6, 2, 33), ((2, 16), 0, 512, 640, 6, 1, 64), ((2, 16), 16, 512, 640, 6, 1, 65),
         ((4, 128), 0, 256, 896, 8, 2, 128), ((4, 128), 2, 256, 896, 8, 2, 129), ((3, 64), 0, 256, 576, 16, 4, 100), ((4, 128), 0, 256, 640, 3, 3, 33),
         ((4, 64), 0, 1600, 1408, 8, 2, 20), ((2, 16), 0, 256, 640, 4, 2, 400)]


# GEMV kernels only: every format with entries of two tokens (two tokens, or no more pairs than experts, or rows of two and of four chunks a
# lane) and of four, rows of w1/w3 of one, two and four chunks a lane, of w2 of one wave and of two, and as many pairs as are queued.
GEMV = [((4, 64), 0, 4096, 2304, 8, 2, 2), ((4, 64), 0, 4096, 2304, 8, 2, 3), ((4, 64), 0, 4096, 2304, 8, 2, 5), ((4, 64), 0, 8192, 640, 8, 2, 7),
        ((4, 64), 0, 1024, 2304, 13, 2, 32), ((4, 64), 8, 4096, 2304, 8, 2, 2), ((4, 64), 8, 4096, 2304, 8, 2, 5), ((4, 32), 0, 1024, 2304, 16, 4, 16),
        ((3, 64), 0, 1920, 4160, 8, 2, 2), ((3, 64), 0, 8192, 640, 8, 2, 6), ((3, 64), 0, 1024, 4416, 16, 3, 21), ((3, 64), 128, 1920, 4160, 8, 2, 2),
        ((3, 64), 4, 4096, 640, 8, 2, 5), ((2, 16), 0, 4096, 1984, 8, 2, 2), ((2, 16), 0, 4096, 2304, 8, 2, 5), ((2, 16), 0, 1024, 640, 13, 2, 32),
        ((2, 16), 16, 1920, 4160, 8, 2, 2), ((2, 16), 16, 4096, 4160, 8, 2, 5), ((2, 16), 128, 8192, 640, 8, 2, 6)]


def tokens(kind, Bn, H, seed):
    x = W.hidden_ar1(seed, 1, Bn, H)[0]
    return x if kind == "spread" else x[:1].expand(Bn, H).contiguous()


def apart(model, Bn):
    """Tokens of which no two take the same expert."""
    pool, picked, taken = W.hidden_ar1(75, 1, 64, model.H)[0], [], set()
    for i, (_, idx, _, _) in enumerate(oracle_routing(model, 0, pool.numpy())):
        if len(picked) < Bn and not taken & set(idx):
            picked.append(i)
            taken |= set(idx)
    assert len(picked) == Bn
    return pool[picked].contiguous()


@pytest.mark.parametrize("fmt,sg,H,F,E,K,Bn", CASES)
@pytest.mark.parametrize("kind", ["spread", "alike"])
def test_batches_queued_without_their_routing(fmt, sg, H, F, E, K, Bn, kind):
    """alike: every token takes the same experts, so a few have all pairs and the others none."""
    queued_and_waiting(fmt, sg, H, F, E, K, Bn, kind)


@pytest.mark.parametrize("fmt,sg,H,F,E,K,Bn", GEMV)
@pytest.mark.parametrize("kind", ["spread", "alike", "apart"])
def test_gemv_batches_queued_without_their_routing(fmt, sg, H, F, E, K, Bn, kind):
    """apart: no two tokens share an expert, where a waiting step takes the kernels of one token."""
    if kind == "apart" and Bn * K > E:
        Bn = E // K // 2 + 1
    queued_and_waiting(fmt, sg, H, F, E, K, Bn, kind, 1000)


def queued_and_waiting(fmt, sg, H, F, E, K, Bn, kind, mfma_min_batch=3):
    model = Model(1, H, F, E, K, [fmt], E, 0, 1e-5, max_batch=Bn, seed=71, scale_group=sg, init_policy=1)
    B.moe_ctx_set_option(model.stack.ctx, "mfma_min_batch", mfma_min_batch)
    x = (apart(model, Bn) if kind == "apart" else tokens(kind, Bn, H, 71)).to(model.stack.device)
    out, h, ys, hs = torch.empty_like(x), torch.empty_like(x), [], []
    for routed in (1, 0, 1):
        B.moe_ctx_set_option(model.stack.ctx, "device_routing", routed)
        out.zero_()
        torch.cuda.synchronize()
        model.stack.step_layer(0, x, out, h)
        model.stack.synchronize()
        ys.append((model.stack.read_y(Bn, H).copy().view(np.uint32), out.cpu().numpy().view(np.uint16)))
        hs.append(h.cpu().numpy().view(np.uint16))
    for y, o in ys[1:]:
        assert (y == ys[0][0]).all() and (o == ys[0][1]).all()
    assert (hs[1] == hs[0]).all()
    st = model.stack.stats()[0]
    routing = oracle_routing(model, 0, x.cpu().numpy())
    assert st["steps"] == 3 and st["steps_device_routed"] == 2 and st["misses"] == 0
    assert st["needed"] == st["hits"] == 3 * len({e for _, idx, _, _ in routing for e in idx})
    worst = 0.0
    for b in sorted({0, 1, Bn // 2, Bn - 1}):
        hb, idx, w, _ = routing[b]
        assert (hs[0][b] == hb.view(np.uint16)).all()
        worst = max(worst, check_y(ys[0][0].view(np.float32)[b], oracle_y(model, 0, hb, idx, w, O.expert_ffn), f"b={b}")[1])
    say(f"routed {fmt} {sg} {H}x{F} E={E} K={K} B={Bn} {kind}: rel {worst:.2e}")
    model.close()


def test_stacks_of_batches_and_tokens():
    """Two layers of different formats, one and several tokens in turn, waiting steps in between: recency and counters as with every
    step waiting."""
    runs = []
    for routed in (1, 0):
        model = Model(2, 256, 512, 8, 2, [(4, 64), (3, 64)], 8, 1, 1e-5, max_batch=40, seed=72, init_policy=1)
        B.moe_ctx_set_option(model.stack.ctx, "device_routing", routed)
        xs = W.hidden_ar1(72, 9, 40, 256).to(model.stack.device)
        outs = []
        for t, n in enumerate((1, 40, 2, 1, 13, 40, 3, 1, 5)):
            x = xs[t, :n].contiguous()
            out = torch.empty_like(x)
            torch.cuda.synchronize()
            if t % 3 == 2:
                model.stack.step_layer(0, x, out, None, B.StepTrace())
            else:
                model.stack.step(x, out)
            outs.append(out)
        model.stack.synchronize()
        st = model.stack.stats()
        routed_steps = [s.pop("steps_device_routed") for s in st]
        assert all(r > 0 for r in routed_steps) if routed else not any(routed_steps)
        runs.append((st, [B.moe_layer_cache_state(l, 8) for l in model.stack.layers], [o.cpu().numpy().view(np.uint16) for o in outs]))
        model.close()
    assert runs[0][0] == runs[1][0] and runs[0][1] == runs[1][1]
    assert all((a == b).all() for a, b in zip(runs[0][2], runs[1][2]))


@pytest.mark.parametrize("fmt,Bn,low", [((3, 64), 4, 1000), ((4, 64), 8, 3), ((3, 64), 40, 3)])
@pytest.mark.parametrize("kind", ["spread", "alike"])
def test_profiled_bytes_are_the_waiting_steps(fmt, Bn, low, kind):
    """Every expert a launch touches counts once: GEMV, 16-token and tile kernels."""
    model = Model(1, 256, 512, 8, 2, [fmt], 8, 0, 1e-5, max_batch=Bn, seed=74, init_policy=1)
    B.moe_ctx_set_option(model.stack.ctx, "mfma_min_batch", low)
    x = tokens(kind, Bn, 256, 74).to(model.stack.device)
    out, got = torch.empty_like(x), []
    for routed in (1, 0):
        B.moe_ctx_set_option(model.stack.ctx, "device_routing", routed)
        B.moe_ctx_profile_enable(model.stack.ctx, True)
        torch.cuda.synchronize()
        model.stack.step_layer(0, x, out)
        p = B.moe_ctx_profile_read(model.stack.ctx)
        got.append([(k.launches, k.bytes) for k in (p.w13, p.w2)])
    model.close()
    assert got[0] == got[1] and all(b > 0 for _, b in got[0])
