"""The large tile kernel in one half of a layer and the 32-token one in the other, against the CPU oracle."""
import pytest

import workload as W
from paper_2312_17238_amd import binding as B

from harness import Model
from test_gpu_tile import one_step, run

pytestmark = pytest.mark.gpu

FORMATS = [((4, 64), 0), ((4, 64), 16), ((4, 128), 2), ((3, 64), 0), ((3, 64), 4), ((2, 16), 0), ((2, 16), 8)]


# Wide: w1/w3 have rows enough for the large kernel, w2 has not; tall: the other way (two-level 2-bit codes take the large one in
# both).  Tokens of an expert: around 52, 105 and 250, one to three tiles a wave and two token blocks.  Contractions of two sets of
# units, the last one short.
@pytest.mark.parametrize("fmt,sg", FORMATS)
@pytest.mark.parametrize("H,F,K,Bn", [(384, 4096, 1, 420), (384, 4096, 2, 420), (384, 4096, 2, 1000),
                                      (8192, 384, 1, 420), (4224, 384, 2, 420), (4224, 384, 2, 1000)])
def test_one_half_large(fmt, sg, H, F, K, Bn):
    run(fmt, sg, H, F, 8, K, 8, Bn, rows={0, Bn // 2, Bn - 1})


@pytest.mark.parametrize("H,F,K,Bn", [(384, 4096, 2, 420), (8192, 384, 1, 420)])
def test_the_halves_do_differ(H, F, K, Bn):
    """The plan's kernels give neither the bits of the large kernel in both halves nor those of the 32-token one."""
    model = Model(1, H, F, 8, K, [(3, 64)], 8, 0, 1e-5, max_batch=Bn, seed=61)
    x = W.hidden_ar1(61, 1, Bn, H)[0].to(model.stack.device)
    ys = []
    for tile in (0, 32, 192):
        B.moe_ctx_set_option(model.stack.ctx, "tile_tokens", tile)
        ys.append(one_step(model, x, 6))
    model.close()
    assert (ys[0] != ys[1]).any() and (ys[0] != ys[2]).any()
