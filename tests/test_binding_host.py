"""The Python binding on the host (no GPU): how it is loaded, and how threads
inside it end."""

from __future__ import annotations

import os
import subprocess
import sys

import pytest
import torch

import paper_1712_02616_amd as iabn
from paper_1712_02616_amd import build as iabn_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# A daemon thread is inside the native call (in an argument's __index__) when
# the interpreter ends, and wakes while it does.
AT_EXIT = """
import importlib.util, sys, threading, time
import torch
spec = importlib.util.spec_from_file_location(sys.argv[1], sys.argv[2])
binding = importlib.util.module_from_spec(spec)
spec.loader.exec_module(binding)
inside = threading.Event()
class Op:
    def __index__(self):
        inside.set()
        time.sleep(1.0)
        return 0
class Last:
    def __del__(self, sleep=time.sleep):
        sleep(2.0)
threading.Thread(target=lambda: binding.call(1, Op()), daemon=True).start()
inside.wait()
last = Last()
"""


def test_a_thread_ends_with_the_interpreter():
    lib = iabn_build.binding_lib()
    if not os.path.exists(lib):
        iabn_build.build_binding()
    res = subprocess.run([sys.executable, "-c", AT_EXIT, "paper_1712_02616_amd._binding", lib],
                         capture_output=True, text=True, cwd=ROOT, timeout=120)
    assert res.returncode == 0, (res.returncode, res.stderr[-500:])


@pytest.mark.parametrize("what", ["not a library", "not built"])
def test_calls_go_on_without_the_fast_path(what, tmp_path, monkeypatch):
    path = tmp_path / "_binding.so"
    if what == "not a library":
        path.write_bytes(b"something else")
    else:
        def no_compiler():
            raise RuntimeError("no compiler")
        monkeypatch.setattr(iabn_build, "build_binding", no_compiler)
    monkeypatch.setattr(iabn_build, "binding_lib", lambda: str(path))
    monkeypatch.setattr(iabn, "_call", iabn._first_call)
    x, c = torch.zeros(2, 3, 4), torch.zeros(3)
    with pytest.warns(RuntimeWarning, match="fast path"):
        with pytest.raises(ValueError, match="HIP device"):
            iabn.iabn_forward_eval(x, c, c, c, c)
    with pytest.raises(ValueError, match="HIP device"):
        iabn.iabn_forward_eval(x, c, c, c, c)


def test_the_fast_path_belongs_to_one_torch(monkeypatch):
    here = iabn_build.binding_lib()
    monkeypatch.setattr(torch, "__version__", "0.0.1")
    assert iabn_build.binding_lib() != here
