"""The gate of more tokens than fit the chip at once, whose blocks take two threads' slices a thread: the bits of h and of the logits, the
selection and the weights are those of the same tokens in steps of a size that the other blocks take."""
import numpy as np
import pytest
import torch

import workload as W
from paper_2312_17238_amd import binding as B

from harness import Model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [64, 1984, 2048, 2112, 4096, 4160, 8192])
@pytest.mark.parametrize("E,eps", [(8, 1e-5), (5, 0.0)])
def test_same_bits_as_few_tokens(H, E, eps):
    """Widths around the slices of 2048 and 4096; 640 tokens against 128 at a time.  Nothing is rounded differently, so every bit agrees."""
    Bn, part = 640, 128
    model = Model(1, H, 64, E, 2, [(4, 64)], E, 0, eps, max_batch=Bn, seed=93)
    x = W.hidden_ar1(93, 1, Bn, H)[0].to(model.stack.device)

    def step(lo, hi):
        h, out, tr = torch.empty_like(x[lo:hi]), torch.empty_like(x[lo:hi]), B.StepTrace()
        torch.cuda.synchronize()
        model.stack.step_layer(0, x[lo:hi], out, h, tr)
        model.stack.synchronize()
        return h.cpu().numpy().view(np.uint16), tr.routing(), np.array(tr.weights()), np.array(tr.logits[: (hi - lo) * E])

    h, idx, w, z = step(0, Bn)
    few = [step(i, i + part) for i in range(0, Bn, part)]
    assert (h == np.concatenate([f[0] for f in few])).all()
    assert idx == sum((f[1] for f in few), [])
    assert (w.reshape(Bn, -1) == np.concatenate([f[2].reshape(part, -1) for f in few])).all()
    assert (z == np.concatenate([f[3] for f in few])).all()
    model.close()
