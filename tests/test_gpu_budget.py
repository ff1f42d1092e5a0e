"""A context holds no more device memory than its budget."""
import re

import numpy as np
import pytest

from paper_2107_01715_amd import workload as W

pytestmark = pytest.mark.gpu


def _search(lib, budget, prec):
    ep = W.env_params(7)
    ctx = lib.Context(0, budget)
    ctx.set_env(ep.delta, ep.vel)
    ctx.set_qnet(W.qnet_blob(W.qnet_weights(7)))
    ctx.set_precision(prec)
    pos, stacks = W.roots(3, 4)
    try:
        ctx.search(pos, stacks, 3, 6, 0.99, lib.correction(True))
    except lib.BctsError:
        ctx.close()                                         # another live context would need a hardware queue of its own
        raise
    return ctx


@pytest.mark.parametrize("prec", ["FP32", "BF16", "FP8"])
def test_the_smallest_budget_is_kept(prec):
    """The refusal names the bytes a search needs; with that budget it runs,
    and what the device then holds more is within it, up to two allocations
    rounded up to 2 MB each."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2107_01715_amd import bcts as lib
    prec = getattr(lib, prec)
    _search(lib, 0, prec).close()                           # the library's own first-use memory
    with pytest.raises(lib.BctsError) as e:
        _search(lib, 1, prec)
    assert e.value.status == lib.E_NOMEM
    need = int(re.search(r"needs (\d+) bytes", str(e.value)).group(1))
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info(0)[0]
    ctx = _search(lib, need, prec)
    held = before - torch.cuda.mem_get_info(0)[0]
    ctx.close()
    assert held <= need + (4 << 20), (held, need)


def test_calibration_in_the_smallest_budget():
    """The FP8 scales come from the FP32 weights, which lie in host memory and
    are copied beside the calibration's plan where there is room."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2107_01715_amd import bcts as lib
    stacks = W.roots(5, 40)[1]

    def scales(budget):
        ctx = lib.Context(0, budget)
        ctx.set_qnet(W.qnet_blob(W.qnet_weights(7)))
        ctx.calibrate_fp8(stacks)
        out = np.array(ctx.get_fp8_scales())
        ctx.close()
        return out

    with pytest.raises(lib.BctsError) as e:
        scales(1)
    assert e.value.status == lib.E_NOMEM
    need = int(re.search(r"needs (\d+) bytes", str(e.value)).group(1))
    assert np.array_equal(scales(need), scales(0))
