"""The large tile kernel in one half of a layer and the 32-token one in the other, against the CPU oracle."""
import pytest

from test_gpu_tile import run

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
