"""The sibling kernel (leaves as positions: a group's background plus what each
child's agent square changes) against the group kernel on rendered frames.

An uncorrected search's root vector is max over a block of r + gamma^d V with
V the largest Q of each leaf.  The leaves' stacks, rendered by the oracle's
environment, go through ``bcts_debug_qnet_siblings``, which takes frames; both
kernels run the same matrix instructions on the same operands, so V has the
same bits and the vectors differ at most by the rounding of the last sum (its
product fused or not): 2 ulp of its largest term.  The roots put the agent at
every column and row, the wrapping ones included.
"""
import numpy as np
import pytest

from oracle import env as E
from paper_2107_01715_amd import workload as W

pytestmark = pytest.mark.gpu
GAMMA = 0.99


@pytest.fixture(scope="module")
def lib():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2107_01715_amd import bcts
    return bcts


def leaves(ep, pos, stack, A, d):
    """(stacks [A^d][4][84][84], returns [A^d]) in the index order of Alg. 1."""
    cur = [(pos.astype(np.int64), stack, 0.0)]
    for k in range(d):
        nxt = []
        for p, s, ret in cur:
            for a in range(A):
                p2, s2, r = E.step(p, s, a, ep.delta, ep.vel)
                nxt.append((p2, s2, ret + GAMMA ** k * r))
        cur = nxt
    return np.array([s for _, s, _ in cur]), np.array([r for _, _, r in cur])


@pytest.mark.parametrize("prec", ["BF16", "FP8"])
@pytest.mark.parametrize("A,d,n", [(1, 1, 3), (2, 1, 84), (18, 1, 14), (3, 2, 9), (18, 2, 1), (2, 4, 2)])
def test_leaves_equal_rendered_frames(lib, prec, A, d, n):
    ep = W.env_params(31 + A)
    ctx = lib.Context(0)
    ctx.set_env(ep.delta, ep.vel)
    ctx.set_qnet(W.qnet_blob(W.qnet_weights(7)))
    pos, stacks = W.roots(1300 + A, n)
    i = np.arange(n)
    pos[:, 0, 0] = (i * 84 // n) % 84                       # the agent: every column, every row
    pos[:, 0, 1] = (83 - i * 37) % 84
    pos[:, 1] = (pos[:, 0] + 2) % 84                        # and a sprite it overlaps
    if prec == "FP8":
        ctx.calibrate_fp8(W.roots(5, 8)[1])
    ctx.set_precision(getattr(lib, prec))
    act, q = ctx.search(pos, stacks, d, A, GAMMA, lib.correction(False))
    want = np.empty((n, A))
    for r in range(n):
        st, ret = leaves(ep, pos[r], stacks[r], A, d)
        v = ctx.debug_qnet_siblings(st, A, A).max(1).astype(np.float64)
        want[r] = (ret + np.float64(np.float32(GAMMA ** d)) * v).reshape(A, -1).max(1)
    tol = 2 * 2.0 ** -23 * max(np.abs(want).max(), 1.0)
    assert np.abs(q - want).max() <= tol, (np.abs(q - want).max(), tol, np.argwhere(np.abs(q - want) > tol)[:8])
    assert np.array_equal(act, q.argmax(1))
    ctx.close()
