"""The scales of the FP32 network's split form (csrc/split_scales.cpp), built on
its own with g++ and checked on the CPU: the operands' planes are formed with
them as the kernels form them, the sums taken in 64 bits, and the result
compared with the network in 64 bits.

Tolerance: operands of 22 bits and a product of 2^-22 left out add at most some
2^-22 of its values a layer; four layers stay within 2^-20 of the largest |Q|.
A network that the rule turns down runs on the FP32 instruction."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2107_01715_amd import workload as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LAYERS = ("conv1", "conv2", "conv3", "fc1")
CHANNELS, SIZES, LOW = (256, 32, 64, 64), (32, 64, 64, 512), 2048.0
FP = ctypes.POINTER(ctypes.c_float)


@pytest.fixture(scope="module")
def scales(tmp_path_factory):
    """weights -> None (turned down) or per layer (row, col, out, bias) scales."""
    if shutil.which("g++") is None:
        pytest.skip("no host C++ compiler")
    so = str(tmp_path_factory.mktemp("split") / "libsplit.so")
    src = [os.path.join(ROOT, "tests", "host", "split_scales_shim.cpp"),
           os.path.join(ROOT, "paper_2107_01715_amd", "csrc", "split_scales.cpp")]
    r = subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-Wextra", "-fsanitize=undefined",
                        *src, "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    fn = ctypes.CDLL(so).shim_split_scales

    def run(weights):
        w = np.concatenate([_rows(weights, n).ravel() for n in LAYERS]).astype(np.float32)
        b = np.concatenate([weights[n + ".b"] for n in LAYERS]).astype(np.float32)
        res = [np.zeros(k, np.float32) for k in (sum(SIZES), sum(CHANNELS), sum(SIZES), sum(SIZES))]
        if not fn(*(x.ctypes.data_as(FP) for x in (w, b, *res))):
            return None
        cut = [np.split(x, np.cumsum(s)[:-1]) for x, s in zip(res, (SIZES, CHANNELS, SIZES, SIZES))]
        return [tuple(c[i] for c in cut) for i in range(4)]

    return run


def _rows(weights, name):
    """[N][K], the input channel innermost (conv1 as it is)."""
    w = np.asarray(weights[name + ".w"], np.float32)
    if name == "conv1":
        return w.reshape(len(w), -1)
    w = w.reshape(len(w), 64, 49) if name == "fc1" else w.reshape(len(w), w.shape[1], -1)
    return np.ascontiguousarray(w.transpose(0, 2, 1)).reshape(len(w), -1)


def _windows(x, side, stride):
    """[n][H][W][C] -> [n][y][x][kh kw c]."""
    v = np.lib.stride_tricks.sliding_window_view(x, (side, side), axis=(1, 2))[:, ::stride, ::stride]
    return v.transpose(0, 1, 2, 4, 5, 3).reshape(*v.shape[:3], -1)


def _inputs(x, layer):
    if layer == 0:
        v = np.lib.stride_tricks.sliding_window_view(x, (8, 8), axis=(2, 3))[:, :, ::4, ::4]
        return v.transpose(0, 2, 3, 1, 4, 5).reshape(len(x), 20, 20, -1)
    return _windows(x, 4, 2) if layer == 1 else _windows(x, 3, 1) if layer == 2 else x.reshape(len(x), -1)


def _exact(weights, stacks):
    x = stacks.astype(np.float64)
    for i, n in enumerate(LAYERS):
        s = _inputs(x, i) @ _rows(weights, n).astype(np.float64).T
        x = np.maximum((s / 255 if i == 0 else s) + weights[n + ".b"], 0)
    return x @ weights["fc2.w"].astype(np.float64).T + weights["fc2.b"]


def _planes(v, low):
    v = v.astype(np.float32)
    hi = v.astype(np.float16)
    assert np.isfinite(hi).all()
    lo = ((v - hi.astype(np.float32)) * np.float32(low)).astype(np.float16)
    return hi.astype(np.float64), lo.astype(np.float64) / low


def _split(weights, stacks, sc):
    x, xl = stacks.astype(np.float64), None
    for i, n in enumerate(LAYERS):
        row, col, out, bias = sc[i]
        w = _rows(weights, n)
        wh, wl = _planes(w * (np.tile(col, w.shape[1] // len(col)) * row[:, None]), 1 if i == 0 else LOW)
        s = _inputs(x, i) @ (wh + wl).T
        if i:
            s = s + _inputs(xl, i) @ wh.T
        y = np.maximum((s.astype(np.float32).astype(np.float64) * out + bias).astype(np.float32), 0)
        x, xl = _planes(y / np.float32(LOW), LOW) if i < 3 else (y.astype(np.float64), None)
    return x @ weights["fc2.w"].astype(np.float64).T + weights["fc2.b"]


def _network(kind):
    w, rng = {k: np.array(v) for k, v in W.qnet_weights(11).items()}, np.random.default_rng(3)
    if kind == "heavy tails":
        for n in LAYERS:
            w[n + ".w"] = (rng.standard_t(4, w[n + ".w"].shape) * w[n + ".w"].std()).astype(np.float32)
    elif kind == "uneven":
        for n, m in zip(LAYERS, LAYERS[1:]):
            k = np.exp2(rng.normal(0, 6, len(w[n + ".b"]))).astype(np.float32)
            w[n + ".w"] *= k.reshape(-1, 1, 1, 1)
            w[n + ".b"] *= k
            w[m + ".w"].reshape(len(w[m + ".w"]), len(k), -1)[...] /= k[:, None]
    elif kind == "sparse":                                  # nine weights in ten are zero, some channels and rows all
        for n in LAYERS:
            w[n + ".w"] *= rng.random(w[n + ".w"].shape) < 0.1
            w[n + ".w"][::7] = 0
        w["conv1.b"][:7] = -0.01
    elif kind == "never fires 2^8" or kind == "never fires 2^36":
        w["conv1.w"][3] *= np.float32(2.0 ** int(kind[14:]))
        w["conv1.b"][3] = -0.75 * np.maximum(w["conv1.w"][3], 0).sum()
    elif kind == "zero":
        for n in LAYERS:
            w[n + ".w"][...] = 0
    elif kind == "far":
        w["conv2.w"] *= np.float32(2.0 ** 80)
        w["conv2.b"] *= np.float32(2.0 ** 80)
        w["conv3.w"] *= np.float32(2.0 ** -80)
    elif kind == "one large weight a row":                  # nothing of the rest would be left beside it
        w["conv2.w"][:, 0, 0, 0] = 2.0 ** 30
    elif kind == "largest":
        w["conv1.w"][...] = 3e38
    return w


@pytest.mark.parametrize("kind,split", [
    ("as drawn", True), ("heavy tails", True), ("uneven", True), ("sparse", True), ("zero", True),
    ("never fires 2^8", True), ("never fires 2^36", False), ("far", False), ("one large weight a row", False),
    ("largest", False)])
def test_networks(scales, kind, split):
    w = _network(kind)
    sc = scales(w)
    assert (sc is not None) == split
    if sc is None:
        return
    stacks = np.concatenate([W.roots(1400, 10)[1], np.zeros((1, 4, 84, 84), np.uint8),
                             np.random.default_rng(1).integers(0, 256, (2, 4, 84, 84), dtype=np.uint8)])
    want = _exact(w, stacks)
    err = np.abs(_split(w, stacks, sc) - want).max(1) / np.abs(want).max(1)
    assert err.max() <= 2.0 ** -20, err


def test_powers_of_two_between_a_channel_and_its_readers_do_not_count(scales):
    """The held weights are the same ones, bit for bit."""
    w, rng = _network("as drawn"), np.random.default_rng(9)
    v = {k: np.array(x) for k, x in w.items()}
    for n, m in zip(LAYERS, LAYERS[1:]):
        k = np.exp2(rng.integers(-20, 21, len(v[n + ".b"]))).astype(np.float32)
        v[n + ".w"] *= k.reshape(-1, 1, 1, 1)
        v[n + ".b"] *= k
        v[m + ".w"].reshape(len(v[m + ".w"]), len(k), -1)[...] /= k[:, None]
    for n, a, b in zip(LAYERS, scales(w), scales(v)):
        held = [_rows(x, n) * (np.tile(s[1], _rows(x, n).shape[1] // len(s[1])) * s[0][:, None]) for x, s in ((w, a), (v, b))]
        assert np.array_equal(*held) and np.array_equal(a[2], b[2]) and np.array_equal(a[3], b[3])
