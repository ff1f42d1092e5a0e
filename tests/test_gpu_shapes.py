"""A root's result does not depend on what is searched with it: levels of few
and of many nodes expand, and roots of few and of many leaves back up, in
launches of different shapes."""
import numpy as np
import pytest

from paper_2107_01715_amd import workload as W

pytestmark = pytest.mark.gpu

# (A, d) of the roots searched together, index of the one also searched alone
BATCHES = [
    ([(9, 3)] + [(2, 3)] * 20, 0),            # 729 leaves among roots of 8
    ([(9, 3)] * 9, 8),                        # levels of 81 and 729 nodes, then 729 and 6,561
    ([(18, 2)] * 13, 12),                     # 4,212 nodes at level 2, 324 alone
    ([(4, 0), (18, 3), (3, 1)], 1),           # depth 0 among deeper ones
]


@pytest.mark.parametrize("shapes,which", BATCHES)
def test_root_alone_and_in_a_batch(shapes, which):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2107_01715_amd import bcts as lib
    ctx = lib.Context(0)
    e = W.env_params(7)
    ctx.set_env(e.delta, e.vel)
    ctx.set_qnet(W.qnet_blob(W.qnet_weights(7)))
    corr = lib.correction(True)
    for prec in (lib.FP32, lib.BF16):
        ctx.set_precision(prec)
        pos, stacks = W.roots(31, len(shapes))
        A = np.array([s[0] for s in shapes], np.int32)
        d = np.array([s[1] for s in shapes], np.int32)
        act, q = ctx.search_batch(pos, stacks, d, A, 0.99, corr)
        one = slice(which, which + 1)
        act1, q1 = ctx.search_batch(pos[one], stacks[one], d[one], A[one], 0.99, corr)
        n = shapes[which][0]
        assert act[which] == act1[0]
        assert np.array_equal(q[which][:n], q1[0][:n])
    ctx.close()


def test_host_inputs_staged_and_direct():
    """36 roots of 28 KB pass through pinned memory in one copy, 40 do not."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2107_01715_amd import bcts as lib
    ctx = lib.Context(0)
    e = W.env_params(7)
    ctx.set_env(e.delta, e.vel)
    ctx.set_qnet(W.qnet_blob(W.qnet_weights(7)))
    ctx.set_precision(lib.BF16)
    pos, stacks = W.roots(32, 40)
    corr = lib.correction(True)
    A, d = np.full(40, 4, np.int32), np.full(40, 2, np.int32)
    act, q = ctx.search_batch(pos, stacks, d, A, 0.99, corr)
    for n in (1, 36, 37):
        act1, q1 = ctx.search_batch(pos[:n], stacks[:n], d[:n], A[:n], 0.99, corr)
        assert np.array_equal(act1, act[:n]) and np.array_equal(q1, q[:n])
    ctx.close()


@pytest.mark.parametrize("prec", ["FP32", "BF16"])
@pytest.mark.parametrize("beam,A,d", [(1, 18, 4), (4, 9, 5), (4, 18, 3)])
def test_kept_nodes_rendered_alone(prec, beam, A, d):
    """A level whose every root is cut renders its kept nodes after the cut;
    beside a root that is not cut there, all nodes before it."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2107_01715_amd import bcts as lib
    ctx = lib.Context(0)
    e = W.env_params(7)
    ctx.set_env(e.delta, e.vel)
    ctx.set_qnet(W.qnet_blob(W.qnet_weights(7)))
    ctx.set_precision(getattr(lib, prec))
    ctx.set_beam(beam)
    corr = lib.correction(True)
    pos, stacks = W.roots(33, 4)
    As, ds = np.full(4, A, np.int32), np.full(4, d, np.int32)
    act, q = ctx.search_batch(pos, stacks, ds, As, 0.99, corr)
    As[3], ds[3] = 1 if beam == 1 else 2, d                 # blocks of at most `beam` nodes at levels 2 and 3: uncut
    if beam == 1:
        corr = lib.correction(False)
        act, q = ctx.search_batch(pos[:3], stacks[:3], ds[:3], As[:3], 0.99, corr)
    act2, q2 = ctx.search_batch(pos, stacks, ds, As, 0.99, corr)
    assert np.array_equal(act2[:3], act[:3]) and np.array_equal(q2[:3, :A], q[:3, :A])
    ctx.close()
