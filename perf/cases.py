"""The work this framework is used for, as cases that can be timed and compared.

A user of the library searches root states of the sprite world (or of the
learned forward model) through the C ABI's Python binding: one root while an
agent plays, a batch of roots while many agents play or a policy is
evaluated, a captured graph for a fixed batch, a served stream of requests.
``listed`` names the cases, ``draw`` gives more of the same ranges, ``prepare``
makes what a program holds before the call (inputs on the device, a context
with its weights), ``run`` is one call, ``exact`` the same values in 64 bits
by plain torch, and ``work`` what a call cannot do without.

Fields of a case: ``world`` "sprite" or "mlp"; ``call`` the entry point;
``precision``; ``roots``; ``actions`` and ``depth`` (0 actions: a mix of 4, 6
and 18 actions and depths 1..``depth``, every root its own); ``penalty`` "eq6",
"gev" or "none"; ``beam`` (0: exhaustive).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2107_01715_amd import bcts, workload as W

GAMMA = float(np.float32(0.99))
WEIGHT_SEED, CALIBRATION_SEED = 7, 2003
FRAME, STATE, MAX_A = 84, 100, 18
PRECISION = {"fp32": bcts.FP32, "bf16": bcts.BF16, "fp8": bcts.FP8}
BYTES = {"fp32": 4, "bf16": 2, "fp8": 1}
# multiply-adds of one dense forward of the value network without its last layer
NET_MACS = 400 * 32 * 256 + 81 * 64 * 512 + 49 * 64 * 576 + 512 * 3136
# stacks a drawn case may evaluate: the cost of the largest listed case
MOST_STACKS = {"bf16": 1_300_000, "fp8": 1_300_000, "fp32": 120_000}
MOST_MLP_NODES = 6_500_000


def _case(name, call, precision, roots, actions, depth, penalty="eq6", beam=0, world="sprite"):
    return {"name": name, "world": world, "call": call, "precision": precision, "roots": roots, "actions": actions,
            "depth": depth, "penalty": penalty, "beam": beam}


def listed():
    return [
        # The benchmark's batch: 256 roots, the full Atari action set, depth 3.
        _case("batch_bf16_18x3", "device", "bf16", 256, 18, 3),
        # The same batch in e4m3, the precision for the highest leaf rate.
        _case("batch_fp8_18x3", "device", "fp8", 256, 18, 3),
        # The working size in full precision: 256 roots of a 6-action game.
        _case("batch_fp32_6x3", "device", "fp32", 256, 6, 3),
        # Roots of different games and depths in one captured launch sequence.
        _case("mixed_graph_bf16", "graph", "bf16", 1032, 0, 3),
        # A deeper tree cut to the best 16 nodes per root action and level.
        _case("beam16_bf16_18x4", "device", "bf16", 64, 18, 4, beam=16),
        # Depth 0: the agent's own Q-values for a batch of states, an odd count.
        _case("policy_bf16_1501", "device", "bf16", 1501, 18, 0, penalty="none"),
        # One decision of one agent, large tree, inputs already on the GPU.
        _case("one_bf16_18x3", "device", "bf16", 1, 18, 3),
        # One decision in full precision from host buffers.
        _case("one_host_fp32_6x3", "host", "fp32", 1, 6, 3),
        # The smallest decision: 4 actions looked ahead once, host buffers.
        _case("one_host_bf16_4x1", "host", "bf16", 1, 4, 1),
        # A burst of requests of mixed shapes through the serving engine.
        _case("serve_burst_bf16", "serve", "bf16", 48, 0, 4),
        # The learned forward model, a batch of 64 roots.
        _case("mlp_batch_10x5", "device", "fp32", 64, 10, 5, world="mlp"),
        # The learned forward model, one binary-action decision.
        _case("mlp_one_2x10", "device", "fp32", 1, 2, 10, world="mlp"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: entry point, precision, actions, depth and options at
    random, then a number of roots spread over the logarithm of what the
    largest listed case would allow."""
    kind = rng.choice(["batch", "batch", "one", "mixed", "beam", "policy", "serve", "mlp", "mlp"])
    penalty = rng.choice(["eq6", "eq6", "gev", "none"])
    if kind == "mlp":
        a = rng.choice([2, 3, 6, 10, 18])
        deepest = int(math.log(MOST_MLP_NODES / 2) / math.log(a))
        d = rng.randint(1, min(12, deepest))
        most = max(1, min(512, MOST_MLP_NODES // sum(a ** k for k in range(1, d + 1))))
        return _unnamed("device" if rng.random() < 0.7 else "host", "fp32", _log_int(rng, 1, most), a, d, penalty, 0,
                        "mlp")
    precision = rng.choice(["bf16", "bf16", "fp8", "fp32"])
    if kind == "policy":
        return _unnamed(rng.choice(["device", "host"]), precision, _log_int(rng, 1, 4000), rng.choice([4, 6, 18]), 0,
                        "none", 0)
    if kind == "serve":
        return _unnamed("serve", precision, _log_int(rng, 1, 64), 0, rng.randint(1, 4), penalty, 0)
    if kind == "mixed":
        return _unnamed(rng.choice(["device", "graph"]), precision,
                        _log_int(rng, 2, 900 if precision != "fp32" else 110), 0, 3, penalty, 0)
    if kind == "beam":
        a = rng.choice([6, 9, 18])
        beam = rng.choice([1, 4, 16, 50])
        case = _unnamed("device", precision, 1, a, rng.randint(3, 5), penalty, beam)
    else:
        a = rng.choice([2, 3, 4, 6, 9, 18])
        deepest = min(5, int(math.log(MOST_STACKS[precision] / 3) / math.log(a)))
        case = _unnamed(rng.choice(["device", "device", "host", "graph"]), precision, 1, a, rng.randint(1, deepest),
                        penalty, 0)
        if kind == "one":
            if a ** case["depth"] < 4000 and rng.random() < 0.4:
                case["call"] = "noalloc"
            return case
    stacks, _ = _counts(case)
    return {**case, "roots": _log_int(rng, 1, max(1, min(1000, MOST_STACKS[precision] // stacks)))}


def _unnamed(*fields):
    case = _case("", *fields)
    del case["name"]
    return case


# ---- shapes ---------------------------------------------------------------
def _shapes(case, seed):
    """(actions, depth) of every root; a mix of shapes comes from the seed."""
    n = case["roots"]
    if case["actions"]:
        return np.full(n, case["actions"], np.int32), np.full(n, case["depth"], np.int32)
    if case["call"] != "serve":
        return W.mixed_shapes(seed, n, d_choices=tuple(range(1, case["depth"] + 1)))
    _, a, d = W.request_arrivals(seed, 1000.0, 1e9, max_requests=n)
    return a, np.minimum(d, case["depth"]).astype(np.int32)


def _tree(a, d, beam):
    """Nodes per level 1..d of one root."""
    out, kept = [], 1
    for k in range(1, d + 1):
        count = kept * a
        out.append(count)
        kept = a * beam if beam and 2 <= k <= d - 1 and count // a > beam else count
    return out


def _counts(case, seed=1):
    """(stacks through the network, expanded nodes) of one pass.  The shapes
    of a mix follow the seed; another seed's mix differs by a few per cent."""
    stacks = nodes = 0
    for a, d in zip(*_shapes(case, seed)):
        levels = _tree(int(a), int(d), case["beam"])
        nodes += sum(levels)
        stacks += levels[-1] if levels else 1
        if levels and case["penalty"] != "none":
            stacks += 1 + (int(a) if d >= 2 else 0)
    return stacks, nodes


def work(case):
    n, out = case["roots"], case["roots"] * 4 * (1 + (case["actions"] or MAX_A))
    if case["world"] == "mlp":
        a, d = case["actions"], case["depth"]
        nodes = n * sum(a ** k for k in range(1, d + 1))
        heads = n * (a ** d + 1 + (a if case["penalty"] != "none" else 0))
        macs = nodes * (3 * STATE * STATE + STATE * (STATE + 1)) + heads * STATE * a
        return {"bytes": 4 * (n * STATE + W.mlp_numel(a)) + out, "flops": 2 * macs}
    stacks, _ = _counts(case)
    # one dense forward per evaluated stack; roots and weights read once
    return {"bytes": n * (4 * FRAME * FRAME + 64) + W.QNET_NUMEL * BYTES[case["precision"]] + out,
            "flops": 2 * stacks * (NET_MACS + 512 * (case["actions"] or 9))}


# ---- what a program holds ---------------------------------------------------
_held = {}


def _context(case):
    """The context of a program with these settings, kept across its calls."""
    key = (case["world"], case["precision"], case["beam"], case["actions"] if case["world"] == "mlp" else 0)
    if key not in _held:
        _held.clear()                       # a program has one; the states of another keep theirs alive
        ctx = bcts.Context(0)
        if case["world"] == "mlp":
            ctx.set_mlp(case["actions"], W.mlp_blob(W.mlp_weights(WEIGHT_SEED, case["actions"]), case["actions"]))
        else:
            env = W.env_params(WEIGHT_SEED)
            ctx.set_env(env.delta, env.vel)
            ctx.set_qnet(W.qnet_blob(W.qnet_weights(WEIGHT_SEED)))
            ctx.set_precision(PRECISION[case["precision"]])
            if case["precision"] == "fp8":
                ctx.calibrate_fp8(W.roots(CALIBRATION_SEED, 32)[1])
            ctx.set_beam(case["beam"])
        _held[key] = ctx
    return _held[key]


class State:
    """Inputs, outputs and the context of one program."""

    def __init__(self, case, seed):
        self.case, self.ctx, self.graph = case, _context(case), None
        self.corr = bcts.correction(case["penalty"] != "none", 1.0,
                                    bcts.CORR_EXACT_GEV if case["penalty"] == "gev" else bcts.CORR_EQ6)
        n, on_gpu = case["roots"], case["call"] in ("device", "noalloc", "graph")
        self.a, self.d = _shapes(case, seed)
        if case["world"] == "mlp":
            self.inputs = (W.mlp_states(seed, n),)
        else:
            self.inputs = W.roots(seed, n)
        if on_gpu:
            self.inputs = tuple(torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in self.inputs)
            self.action = torch.zeros(n, dtype=torch.int32, device="cuda")
            self.q = torch.zeros(n, case["actions"] if case["world"] == "mlp" else MAX_A, device="cuda")
        if case["call"] == "graph":
            self.graph = self.ctx.graph_create(*self.inputs, self.d, self.a, GAMMA, self.corr, self.action, self.q)

    def __del__(self):
        if self.graph is not None:
            self.graph.close()              # before the context it was made from


def prepare(case, seed):
    return State(case, seed)


def run(state):
    s, case, ctx = state, state.case, state.ctx
    if case["world"] == "mlp":
        if case["call"] == "host":
            action, q = ctx.mlp_search(*s.inputs, case["depth"], case["actions"], GAMMA, s.corr)
            return {"action": action, "q": q}
        ctx.mlp_search_device(*s.inputs, case["depth"], GAMMA, s.corr, s.action, s.q)
    elif case["call"] == "host":
        action, q = ctx.search(*s.inputs, case["depth"], case["actions"], GAMMA, s.corr)
        return {"action": action, "q": q}
    elif case["call"] == "serve":
        tickets = [ctx.submit(p, x, int(d), int(a), GAMMA, s.corr) for p, x, a, d in zip(*s.inputs, s.a, s.d)]
        while ctx.progress() > 0:
            pass
        action, q = np.empty(len(tickets), np.int32), np.full((len(tickets), MAX_A), -np.inf, np.float32)
        for i, (ticket, a) in enumerate(zip(tickets, s.a)):
            action[i], q[i, :a], _ = ctx.poll(ticket, int(a))
        return {"action": action, "q": q}
    elif case["call"] == "graph":
        s.graph.launch()
    elif case["call"] == "noalloc":
        ctx.search_batch_device_noalloc(*s.inputs, s.d, s.a, GAMMA, s.corr, s.action, s.q)
    else:
        ctx.search_batch_device(*s.inputs, s.d, s.a, GAMMA, s.corr, s.action, s.q)
    return {"action": s.action, "q": s.q}


# ---- the same in 64 bits ----------------------------------------------------
def exact(case, seed):
    """Root vectors in 64 bits (None for the actions).  A cut tree is ranked by
    32-bit returns, so it has no 64-bit counterpart."""
    if case["beam"]:
        return None
    n = case["roots"]
    shapes_a, shapes_d = _shapes(case, seed)
    wide = case["actions"] if case["world"] == "mlp" or case["call"] == "host" else MAX_A
    q = torch.full((n, wide), -math.inf, dtype=torch.float64, device="cuda")
    if case["world"] == "mlp":
        model = _MlpModel(case["actions"])
        roots = [(s,) for s in torch.from_numpy(W.mlp_states(seed, n)).cuda().double()]
    else:
        model = _SpriteModel()
        pos, stacks = (torch.from_numpy(x).cuda() for x in W.roots(seed, n))
        roots = list(zip(pos.long(), stacks))
    for r in range(n):
        a, d = int(shapes_a[r]), int(shapes_d[r])
        q[r, :a] = _root_vector(model, roots[r], a, d, case["penalty"])
    return {"action": None, "q": q}


def _root_vector(model, root, a, d, penalty):
    level, returns, first = model.start(root), torch.zeros(1, dtype=torch.float64, device="cuda"), None
    q0 = model.values(level, a)[0] if d == 0 or penalty != "none" else None
    if d == 0:
        return q0
    for k in range(d):
        level, reward = model.step(level, a)
        returns = returns.repeat_interleave(a) + GAMMA ** k * reward
        if k == 0 and penalty != "none":
            first = reward + GAMMA * model.values(level, a).amax(1)
    best = model.values(level, a).amax(1)
    out = (returns + GAMMA ** d * best).reshape(a, -1).amax(1)
    if penalty == "none":
        return out
    delta, greedy = (first - q0).abs(), int(q0.argmax())
    others = torch.arange(a, device="cuda") != greedy
    coef_e, coef_o = _penalty(a, d, penalty)
    shift = GAMMA ** d * (coef_e * delta[others].mean() - coef_o * delta[greedy])
    return torch.where(others, out - shift, out)


def _penalty(a, d, penalty):
    if penalty == "eq6":
        root = math.sqrt(math.log(a))
        return root * math.sqrt(d) - 1 / math.sqrt(8), root * math.sqrt(d - 1) - 1 / math.sqrt(8)

    def gap(count):
        if count <= 1:
            return 0.0
        euler, tail = 0.57721566490153286, torch.tensor([1 / (math.e * count), 1 / count], dtype=torch.float64)
        z = -torch.special.ndtri(tail)
        return float(euler * z[0] + (1 - euler) * z[1])

    return gap(a ** d - a ** (d - 1)) / math.sqrt(2), gap(a ** (d - 1)) / math.sqrt(2)


class _SpriteModel:
    CHUNK = 2048

    def __init__(self):
        env = W.env_params(WEIGHT_SEED)
        self.delta, self.vel = (torch.from_numpy(np.asarray(x)).cuda().long() for x in (env.delta, env.vel))
        self.w = {k: torch.from_numpy(v).cuda().double() for k, v in W.qnet_weights(WEIGHT_SEED).items()}

    def start(self, root):
        return root[0][None], root[1][None]

    def step(self, level, a):
        pos, stacks = level
        moved = pos.repeat_interleave(a, 0)
        moved[:, 0] += self.delta[:a].repeat(len(pos), 1)
        moved[:, 1:] += self.vel
        moved %= FRAME
        gap = (moved[:, :1] - moved[:, 1:]) % FRAME
        reward = (torch.minimum(gap, FRAME - gap) < 6).all(2).sum(1).double()
        line = torch.arange(FRAME, device="cuda")
        cover = ((line - moved[..., None]) % FRAME) < 6                    # [nodes][sprite][x, y][84]
        frame = torch.zeros(len(moved), FRAME, FRAME, dtype=torch.uint8, device="cuda")
        for i in list(range(1, 8)) + [0]:
            square = cover[:, i, 1, :, None] & cover[:, i, 0, None, :]
            frame.masked_fill_(square, 255 if i == 0 else 128)
        return (moved, torch.cat([stacks.repeat_interleave(a, 0)[:, 1:], frame[:, None]], 1)), reward

    def values(self, level, a):
        return torch.cat([self._forward(x, a) for x in level[1].split(self.CHUNK)])

    def _forward(self, stacks, a):
        x, w = stacks.double() / 255, self.w
        for name, size, stride, axis in (("conv1", 8, 4, 2), ("conv2", 4, 2, 1), ("conv3", 3, 1, 1)):
            x = x.unfold(axis, size, stride).unfold(axis + 1, size, stride)
            if axis == 2:                                                  # [n][c][y][x][kh][kw] to channels after x
                x = x.permute(0, 2, 3, 1, 4, 5)
            n, side = x.shape[0], x.shape[1]
            kernel = w[name + ".w"].reshape(len(w[name + ".w"]), -1)
            x = torch.addmm(w[name + ".b"], x.reshape(n * side * side, -1), kernel.t()).relu_()
            x = x.reshape(n, side, side, -1)
        x = x.permute(0, 3, 1, 2).reshape(x.shape[0], -1)
        x = torch.addmm(w["fc1.b"], x, w["fc1.w"].t()).relu_()
        return torch.addmm(w["fc2.b"][:a], x, w["fc2.w"][:a].t())


class _MlpModel:
    def __init__(self, a):
        self.w = {k: torch.from_numpy(v).cuda().double() for k, v in W.mlp_weights(WEIGHT_SEED, a).items()}

    def start(self, root):
        return root[0][None]

    def step(self, level, a):
        w = self.w
        x = level @ w["l1.w"][:, :STATE].t() + w["l1.b"]
        x = (x[:, None, :] + w["l1.w"][:, STATE:].t()[None]).reshape(-1, STATE).relu_()
        for name in ("l2", "l3"):
            x = torch.addmm(w[name + ".b"], x, w[name + ".w"].t()).relu_()
        x = torch.addmm(w["out.b"], x, w["out.w"].t())
        return x[:, :STATE].contiguous(), x[:, STATE]

    def values(self, level, a):
        return torch.addmm(self.w["q.b"], level, self.w["q.w"].t())
