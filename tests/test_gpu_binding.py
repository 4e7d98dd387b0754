"""The binding's native fast path against its Python path (an explicit stream
takes the latter): the same bits from every entry point, and the same errors
for the same wrong arguments, whichever path meets them first.
"""

from __future__ import annotations

import ctypes

import pytest
import torch

import paper_1712_02616_amd as iabn

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP GPU")]

C = 6
SHAPES = [(2, C, 5, 7), (3, C, 64), (4, C)]


def _state(shape, dtype):
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    t = {k: torch.randn(shape, generator=g, device="cuda").to(dtype) for k in ("x", "z", "dz")}
    for k in ("gamma", "beta", "rm", "rv", "sm", "sv", "dg", "db"):
        t[k] = torch.rand(C, generator=g, device="cuda") + 0.5
    return t


CALLS = {
    "forward_train": lambda t, **k: iabn.iabn_forward_train(
        t["x"], t["gamma"], t["beta"], t["rm"], t["rv"], t["sm"], t["sv"], 1e-5, 0.1, 0.01, **k),
    "noalloc": lambda t, **k: iabn.iabn_forward_train_noalloc(
        t["x"], t["gamma"], t["beta"], t["rm"], t["rv"], t["sm"], t["sv"], **k),
    "eval": lambda t, **k: iabn.iabn_forward_eval(t["x"], t["gamma"], t["beta"], t["rm"], t["rv"], **k),
    "backward": lambda t, **k: iabn.iabn_backward(
        t["z"], t["dz"], t["gamma"], t["beta"], t["sv"], t["dg"], t["db"], **k),
    "backward_ii": lambda t, **k: iabn.iabn_backward_ii(
        t["z"], t["dz"], t["gamma"], t["beta"], t["sv"], t["dg"], t["db"], **k),
    "std_forward": lambda t, **k: iabn.iabn_std_forward_train(
        t["x"], t["z"], t["gamma"], t["beta"], t["rm"], t["rv"], t["sm"], t["sv"], **k),
    "std_backward": lambda t, **k: iabn.iabn_std_backward(
        t["x"], t["z"], t["dz"], t["gamma"], t["beta"], t["sm"], t["sv"], t["dg"], t["db"], **k),
    "ckpt_forward": lambda t, **k: iabn.iabn_ckpt_forward_train(
        t["x"], t["z"], t["gamma"], t["beta"], t["rm"], t["rv"], t["sm"], t["sv"], **k),
    "ckpt_recompute": lambda t, **k: iabn.iabn_ckpt_recompute(t["x"], t["z"], t["gamma"], t["beta"], **k),
    "ckpt_backward": lambda t, **k: iabn.iabn_ckpt_backward(
        t["x"], t["dz"], t["gamma"], t["beta"], t["sv"], t["dg"], t["db"], **k),
}


@pytest.mark.parametrize("call", CALLS)
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
def test_same_bits(call, dtype):
    for shape in SHAPES:
        a, b = _state(shape, dtype), _state(shape, dtype)
        ra = CALLS[call](a)
        rb = CALLS[call](b, stream=torch.cuda.current_stream())
        torch.cuda.synchronize()
        for k in a:
            assert torch.equal(a[k], b[k]), (shape, k)
        assert any(ra is v for v in a.values()) and torch.equal(ra, rb)


def _wrong(name):
    """The state with one argument that must be refused."""
    t = _state((2, C, 5, 7), torch.float32)
    if name == "not contiguous":
        t["x"] = t["z"] = torch.randn(2, C, 7, 5, device="cuda").transpose(2, 3)
    elif name == "dtype":
        t["x"], t["z"] = t["x"].double(), t["z"].double()
    elif name == "host tensor":
        t["x"], t["z"] = t["x"].cpu(), t["z"].cpu()
    elif name == "one dim":
        t["x"] = t["z"] = torch.randn(C, device="cuda")
    elif name == "not a tensor":
        t["x"] = t["z"] = 3
    elif name == "half parameters":
        t["gamma"] = t["gamma"].half()
    elif name == "short parameters":
        t["gamma"] = t["gamma"][:-1].contiguous()
    elif name == "strided parameters":
        t["gamma"] = torch.rand(2 * C, device="cuda")[::2]
    elif name == "one value per channel":
        for k in ("x", "z", "dz"):
            t[k] = torch.randn(1, C, 1, device="cuda")
    return t


@pytest.mark.parametrize("call", ["forward_train", "backward", "std_forward", "ckpt_recompute", "eval"])
@pytest.mark.parametrize("what", ["not contiguous", "dtype", "host tensor", "one dim", "not a tensor",
                                  "half parameters", "short parameters", "strided parameters",
                                  "one value per channel"])
def test_same_errors(call, what):
    got = []
    for kw in ({}, {"stream": torch.cuda.current_stream()}):
        try:
            CALLS[call](_wrong(what), **kw)
            got.append(None)
        except Exception as e:  # noqa: BLE001
            got.append((type(e), str(e)))
    assert got[0] == got[1]
    if what != "one value per channel" or call in ("forward_train", "backward", "std_forward"):
        assert got[0] is not None


def test_workspace_arguments():
    t = _state((4, C, 20000), torch.float16)
    need = iabn.iabn_workspace_size(4, C, 20000, torch.float16)
    CALLS["forward_train"](t, workspace=torch.empty(need, dtype=torch.uint8, device="cuda"))
    CALLS["forward_train"](t, workspace=torch.empty(need // 4 + 1, device="cuda"))
    with pytest.raises(iabn.IabnError, match="needed"):
        CALLS["forward_train"](t, workspace=torch.empty(need - 16, dtype=torch.uint8, device="cuda"))
    with pytest.raises(ValueError, match="workspace"):
        CALLS["forward_train"](t, workspace=torch.empty(need, dtype=torch.uint8))
    with pytest.raises(iabn.IabnError, match="eps"):
        iabn.iabn_forward_train(t["x"], t["gamma"], t["beta"], t["rm"], t["rv"], t["sm"], t["sv"], eps=0.0)


def test_other_threads_run_meanwhile():
    """The fast path takes its workspace and launches without the GIL: with
    entry points that report the GIL's state in place of the library's, a
    workspace of no bytes is asked for (the address of the thread that holds
    the GIL otherwise, too many to get) and the launch's status is 0."""
    t = _state((2, C, 64), torch.float32)
    CALLS["forward_train"](t)  # loads the fast path
    addr = lambda fn: ctypes.cast(fn, ctypes.c_void_p).value  # noqa: E731
    table = type(iabn.load().table_array)(*iabn.load().table_array)
    table[iabn._WORKSPACE_SIZE] = addr(ctypes.pythonapi._PyThreadState_UncheckedGet)
    table[iabn._FORWARD_TRAIN] = addr(ctypes.pythonapi.PyGILState_Check)
    rc = iabn._call(ctypes.addressof(table), iabn._FORWARD_TRAIN, t["x"], t["gamma"], t["beta"], t["rm"],
                    t["rv"], t["sm"], t["sv"], 1e-5, 0.1, 0.01, None)
    assert rc == 0


def test_current_stream():
    """The fast path runs on torch's current stream."""
    t = _state((8, C, 4096), torch.float32)
    ref = _state((8, C, 4096), torch.float32)
    CALLS["forward_train"](ref)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        x0 = t["x"].clone()
        torch.cuda._sleep(20_000_000)
        t["x"].zero_()
        t["x"].copy_(x0)
        CALLS["forward_train"](t)
    s.synchronize()
    assert torch.equal(t["x"], ref["x"])
