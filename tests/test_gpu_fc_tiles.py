"""fc1's tile sizes (32, 64, 128 and 256 stacks) give a stack the same bits: every
output sums over K in the same order whatever the tile, and fc2 associates its
sum the same way behind each."""
import numpy as np
import pytest

from paper_2107_01715_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("folded", [1, 0])
@pytest.mark.parametrize("prec", ["BF16", "FP8"])
def test_tiles_give_the_same_bits(prec, folded):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2107_01715_amd import bcts as lib
    ctx = lib.Context(0)
    ctx.set_qnet(W.qnet_blob(W.qnet_weights(7)))
    base = W.roots(1400, 150)[1]
    ctx.calibrate_fp8(base[:16])
    ctx.set_precision(getattr(lib, prec))
    ctx.set_tuning(lib.TUNE_FC2_FOLDED, folded)
    stacks = np.tile(base, (340, 1, 1, 1))              # 51,000 stacks: the largest tiles only
    whole = ctx.debug_qnet(stacks, 18)
    for n in (1, 16, 31, 33, 512, 513, 1501, 2048, 2049, 8193, 16385, 32768, 32769, 34900):
        q = ctx.debug_qnet(stacks[:n], 18)
        assert np.array_equal(q, whole[:n]), (n, np.abs(q - whole[:n]).max())
    ctx.close()
