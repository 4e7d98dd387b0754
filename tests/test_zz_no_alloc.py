"""iabn_forward_train_noalloc, the training forward for callers that cannot
allocate (the streaming kernels keep their partials, and the slice-resident
kernels exchange their sums, in the library's static scratch), through the C
ABI against iabn_forward_train with a caller's workspace: the same kernels, so
the outputs must be bit-identical.  Calls in a row on shapes that use the
scratch, one smaller than the one before, then a channel-resident shape (no
scratch), the largest uses of either kind, and the first shape again (the
scratch holds the last call's values, which must not leak into the next)."""

from __future__ import annotations

import ctypes

import pytest
import torch

import paper_1712_02616_amd as iabn
import workloads
from gpu_helpers import TORCH_DTYPES, GpuLayer, say

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP GPU")]

SHAPES = [
    # (N, C, HW, dtype, seed, kernels): large, then smaller
    (3, 32, 20008, "f16", 71, "streaming"),
    (3, 5, 49, "f32", 72, "streaming"),
    (4, 256, 1024, "bf16", 73, "channel-resident"),
    # the most partials per call (765 slices), and nearly the most sums (510)
    (1100, 255, 31, "f16", 75, "streaming"),
    (8, 255, 65536, "f16", 74, "slice-resident"),
    (3, 32, 20009, "f16", 76, "slice-resident"),
    (3, 32, 20008, "f16", 71, "streaming"),
]


def run_noalloc(L: GpuLayer, eps, mom, slope):
    """iabn_forward_train_noalloc through the C ABI (raw pointers, the current stream)."""
    lib = iabn.load()
    N, C, HW = L.shape
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    code = iabn.DTYPE_CODES[L.x.dtype]
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    rc = lib.iabn_forward_train_noalloc(p(L.x), code, p(L.gamma), p(L.beta), p(L.running_mean),
                                        p(L.running_var), p(L.save_mean), p(L.save_var), eps, mom,
                                        slope, N, C, HW, st)
    assert rc == 0, lib.iabn_last_error().decode()


def test_noalloc_equals_workspace_forward():
    eps, mom, slope = 1e-5, 0.1, 0.01
    for N, C, HW, dtype, seed, kernels in SHAPES:
        inp = workloads.make_layer(N, C, HW, dtype, seed, dz_std=0.1, gamma_sign=True)
        plan = iabn.iabn_plan("forward_train", TORCH_DTYPES[dtype], N, C, HW)
        say("noalloc forward %s shape=%s %s" % (dtype, (N, C, HW), kernels))
        assert kernels == ("channel-resident" if plan["channel_resident"] else
                           "slice-resident" if plan["reg_accesses"] else "streaming"), plan
        A = GpuLayer(inp)
        A.forward_train(eps, mom, slope)
        B = GpuLayer(inp)
        run_noalloc(B, eps, mom, slope)
        torch.cuda.synchronize()
        for k in ("x", "save_mean", "save_var", "running_mean", "running_var"):
            assert torch.equal(getattr(A, k), getattr(B, k)), (k, (N, C, HW, dtype))


def test_noalloc_validates_like_the_workspace_forward():
    inp = workloads.make_layer(2, 5, 1000, "f32", 75)
    L = GpuLayer(inp)
    before = L.x.clone()
    say("noalloc error paths")
    with pytest.raises(iabn.IabnError) as e:
        iabn.iabn_forward_train_noalloc(L.x, L.gamma, L.beta, L.running_mean, L.running_var,
                                        L.save_mean, L.save_var, 1e-5, 0.1, 0.0)
    assert e.value.status == 3
    with pytest.raises(iabn.IabnError) as e:
        iabn.iabn_forward_train_noalloc(L.x, L.gamma, L.beta, L.running_mean, L.running_var,
                                        L.save_mean, L.save_var, 1e-5, 1.5, 0.01)
    assert e.value.status == 3
    torch.cuda.synchronize()
    assert torch.equal(L.x, before)
