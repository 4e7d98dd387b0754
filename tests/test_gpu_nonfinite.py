"""Infinities and NaN, on every kernel family: a channel whose variance is
infinite (given to the backward or the inference forward, or from squares
that overflow fp32) has 1/sigma = 0, so its outputs are f(beta) and its
gradients zero, whichever kernels run the shape; a channel that holds an
infinity or a NaN spoils no other channel.
"""

from __future__ import annotations

import pytest
import torch

import paper_1712_02616_amd as iabn
from gpu_helpers import TOL, TORCH_DTYPES, say

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP GPU")]

SLOPE = 0.01
BAD = 2  # the channel
SHAPES = [
    (3, 5, 49),      # streaming
    (2, 16, 64),     # one slice per channel
    (2, 40, 9409),   # slices that exchange sums, ragged rows
    (2, 300, 9409),  # one ragged slice per channel
    (2, 256, 64),    # channel-resident
    (4, 300, 1001),  # channel-resident, narrow accesses
]
ID = lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v)  # noqa: E731


def _params(C):
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    p = {k: torch.rand(C, generator=g, device="cuda") + 0.5 for k in ("gamma", "rm", "rv", "sm", "sv")}
    p["beta"] = torch.randn(C, generator=g, device="cuda")
    p["dg"], p["db"] = torch.empty(C, device="cuda"), torch.empty(C, device="cuda")
    return p


def _randn(shape, dtype, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda").to(TORCH_DTYPES[dtype])


def _forward(kind, x, p):
    """(z, the other stored tensor or None)"""
    a = (p["gamma"], p["beta"], p["rm"], p["rv"])
    if kind == "eval":
        return iabn.iabn_forward_eval(x, *a), None
    a += (p["sm"], p["sv"])
    if kind == "train":
        return iabn.iabn_forward_train(x, *a), None
    z = torch.empty_like(x)
    (iabn.iabn_std_forward_train if kind == "std" else iabn.iabn_ckpt_forward_train)(x, z, *a)
    return z, x


def _backward(kind, u, z, dz, p):
    a = (p["gamma"], p["beta"])
    if kind == "std":
        return iabn.iabn_std_backward(u, z, dz, *a, p["sm"], p["sv"], p["dg"], p["db"])
    fn = {"train": iabn.iabn_backward, "ii": iabn.iabn_backward_ii, "ckpt": iabn.iabn_ckpt_backward}[kind]
    return fn(u, dz, *a, p["sv"], p["dg"], p["db"])


def _f_of_beta(p, dtype):
    y = p["beta"][BAD]
    return (y if y >= 0 else SLOPE * y).to(TORCH_DTYPES[dtype])


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("shape", SHAPES, ids=ID)
def test_infinite_running_variance(shape, dtype):
    say("nonfinite eval %s %s" % (shape, dtype))
    p = _params(shape[1])
    p["rv"][BAD] = float("inf")
    z, _ = _forward("eval", _randn(shape, dtype, 1), p)
    torch.cuda.synchronize()
    assert bool((z[:, BAD] == _f_of_beta(p, dtype)).all())
    assert bool(torch.isfinite(z).all())


@pytest.mark.parametrize("kind", ["train", "ii", "std", "ckpt"])
@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("shape", SHAPES, ids=ID)
def test_infinite_saved_variance(shape, dtype, kind):
    say("nonfinite backward %s %s %s" % (kind, shape, dtype))
    p = _params(shape[1])
    p["sv"][BAD] = float("inf")
    dx = _backward(kind, _randn(shape, dtype, 1), _randn(shape, dtype, 2), _randn(shape, dtype, 3), p)
    torch.cuda.synchronize()
    assert bool((dx[:, BAD] == 0).all())
    for t in (dx, p["dg"], p["db"]):
        assert bool(torch.isfinite(t).all())


@pytest.mark.parametrize("kind", ["train", "std", "ckpt"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=ID)
def test_squares_that_overflow(shape, dtype, kind):
    """A thread that adds several squares in fp32 has an infinite sum, and the
    outputs are f(beta); where every thread has one value its shifted sums are
    zero, the rest is in double, and the outputs are the normalised values."""
    say("nonfinite forward %s %s %s" % (kind, shape, dtype))
    p = _params(shape[1])
    x = _randn(shape, dtype, 1)
    x[:, BAD] *= 1e25
    v = x[:, BAD].double()
    y = (v - v.mean()) / v.std(correction=0) * p["gamma"][BAD] + p["beta"][BAD]
    normalised = torch.where(y >= 0, y, SLOPE * y)
    z, _ = _forward(kind, x, p)
    torch.cuda.synchronize()
    assert p["sv"][BAD] == float("inf") and bool(torch.isfinite(p["sm"]).all())
    assert bool(torch.isfinite(z).all())
    assert bool((z[:, BAD] == _f_of_beta(p, dtype)).all()) or torch.allclose(
        z[:, BAD].double(), normalised, rtol=TOL[dtype], atol=TOL[dtype])


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("shape", SHAPES, ids=ID)
def test_one_value_spoils_its_channel_only(shape, value):
    say("nonfinite value %s %s" % (value, shape))
    N, C, HW = shape
    rest = [c for c in range(C) if c != BAD]
    got = []
    for bad in (False, True):
        p = _params(C)
        x, z, dz = (_randn(shape, "f16", s) for s in (1, 2, 3))
        if bad:
            x[N - 1, BAD, HW // 2] = dz[N - 1, BAD, HW // 2] = value
        _forward("train", x, p)
        _backward("train", z, z, dz, dict(p, sv=torch.ones(C, device="cuda")))
        got.append({"z": x, "dx": dz, "dg": p["dg"], "db": p["db"], "sm": p["sm"], "sv": p["sv"],
                    "rm": p["rm"], "rv": p["rv"]})
    torch.cuda.synchronize()
    for k, v in got[0].items():
        w = got[1][k]
        a, b = (v[:, rest], w[:, rest]) if v.dim() == 3 else (v[rest], w[rest])
        assert torch.equal(a, b), k
    assert not bool(torch.isfinite(got[1]["z"][:, BAD]).any())
    assert not bool(torch.isfinite(got[1]["dx"][:, BAD]).any())
    for k in ("sm", "dg", "db"):
        assert not bool(torch.isfinite(got[1][k][BAD])), k
