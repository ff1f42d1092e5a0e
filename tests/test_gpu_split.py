"""The FP32 network in split FP16: a stack's values do not depend on the batch
(which kernels, tiles and runs it goes through), and lie as close to 64 bits as
the split allows."""
import numpy as np
import pytest

from paper_2107_01715_amd import workload as W

pytestmark = pytest.mark.gpu


def _lib():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2107_01715_amd import bcts as lib
    return lib


def _exact(weights, stacks):
    """Q in float64 by plain torch on the CPU."""
    import torch
    import torch.nn.functional as F
    w = {k: torch.from_numpy(np.asarray(v)).double() for k, v in weights.items()}
    x = torch.from_numpy(stacks).double() / 255.0
    x = F.relu(F.conv2d(x, w["conv1.w"], w["conv1.b"], stride=4))
    x = F.relu(F.conv2d(x, w["conv2.w"], w["conv2.b"], stride=2))
    x = F.relu(F.conv2d(x, w["conv3.w"], w["conv3.b"]))
    x = F.relu(F.linear(x.flatten(1), w["fc1.w"], w["fc1.b"]))
    return F.linear(x, w["fc2.w"], w["fc2.b"]).numpy()


def test_bits_do_not_depend_on_the_batch():
    lib = _lib()
    ctx = lib.Context(0)
    ctx.set_qnet(W.qnet_blob(W.qnet_weights(7)))
    ctx.set_precision(lib.FP32)
    base = W.roots(1400, 162)[1]
    base[:, :3] = np.repeat(base[::18, :3], 18, axis=0)     # siblings: 9 groups of 18 share channels 0..2
    stacks = np.tile(base, (102, 1, 1, 1))                  # 16,524 stacks
    whole = ctx.debug_qnet(stacks, 18)
    for n in (1, 2, 31, 33, 161, 768, 769, 1023, 1025, 13000, 16384, 16385):
        q = ctx.debug_qnet(stacks[:n], 18)
        assert np.array_equal(q, whole[:n]), (n, np.abs(q - whole[:n]).max())
    for n, group in ((18, 18), (162, 18), (162, 3), (1026, 18), (1026, 2), (1026, 9), (16524, 18), (16524, 6)):
        q = ctx.debug_qnet_siblings(stacks[:n], 18, group)
        assert np.array_equal(q, whole[:n]), (n, group, np.abs(q - whole[:n]).max())
    ctx.close()


@pytest.mark.parametrize("scale", [1.0, 2.0 ** 9, 2.0 ** -12, 2.0 ** 80])
def test_against_64_bits(scale):
    """Layer weights of very different sizes (2^80: on the FP32 instruction).  Operands carry 22 bits and the
    smallest product is left out (2^-22): 3 x 2^-22 of a layer's absolute sum
    at most, some 2^-20 of its result where half of the sum cancels; four
    layers and fc2: 2^-18."""
    lib = _lib()
    weights = dict(W.qnet_weights(11))
    weights["conv2.w"] = (weights["conv2.w"] * np.float32(scale)).astype(np.float32)
    weights["conv3.w"] = (weights["conv3.w"] / np.float32(scale)).astype(np.float32)
    weights["conv2.b"] = (weights["conv2.b"] * np.float32(scale)).astype(np.float32)
    ctx = lib.Context(0)
    ctx.set_qnet(W.qnet_blob(weights))
    ctx.set_precision(lib.FP32)
    stacks = W.roots(1400, 40)[1]
    q = ctx.debug_qnet(stacks, 18)
    want = _exact(weights, stacks)
    assert np.abs(q - want).max() <= 2.0 ** -18 * np.abs(want).max()
    ctx.close()
