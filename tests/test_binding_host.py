"""The Python binding on the host (no GPU): how it is loaded, and how threads
inside it end."""

from __future__ import annotations

import os
import subprocess
import sys

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
    iabn.load()
    res = subprocess.run([sys.executable, "-c", AT_EXIT, "paper_1712_02616_amd._binding",
                          iabn_build.BINDING_LIB], capture_output=True, text=True, cwd=ROOT, timeout=120)
    assert res.returncode == 0, (res.returncode, res.stderr[-500:])
