"""The slice-resident kernels at the sizes where they can go wrong: each rung
of registers and what lies past it, tiles of whole rows and of parts of rows,
ragged rows with every tail, unaligned tensors, channels cut into slices that
exchange their sums (also when blocks give up waiting, in a library built to
abandon every other slice), workspaces full of garbage, graph replays and
concurrent streams.  Each shape goes through the parity checks of
test_gpu_random_shapes.py (oracle, guard bands), InPlace-ABN I and II and both
comparison blocks.
"""

from __future__ import annotations

import ctypes
import os

import numpy as np
import pytest
import torch

import oracle
import paper_1712_02616_amd as iabn
import test_gpu_graph
import test_gpu_random_shapes as parity
import test_gpu_streams
import workloads
from gpu_helpers import TORCH_DTYPES, assert_close, say, to_f64
from paper_1712_02616_amd import build as iabn_build

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a HIP GPU")]


def _shape(N, C, HW, dtype, offset=0):
    name = "%s_n%d_c%d_hw%d_o%d" % (dtype, N, C, HW, offset)
    return parity.Shape(name, N, C, HW, dtype, offset, 9000 + (N * 31 + C * 7 + HW) % 1000)


# One row of J * 1024 + 1 fp32 values in 257 channels: one slice of J 16-byte
# accesses per thread (the last ones of each rung, and the first past it).
RUNGS = [_shape(1, 257, J * 1024 + 1, "f32") for J in (4, 5, 9, 17, 21, 25, 33, 51)]
# Tails of 1 to 7 elements, tiles of parts of rows.
TAILS = [_shape(3, 40, 2048 + k, dt) for dt, ks in (("f16", (1, 2, 3, 5, 6, 7)), ("f32", (1, 3)))
         for k in ks]
SMALL = [
    _shape(2, 16, 64, "f32"),           # less than a tile
    _shape(100, 300, 71, "f16"),        # whole rows per tile, the last tile with fewer; long tails
    _shape(37, 270, 115, "bf16"),
    _shape(5, 7, 1041, "bf16"),
    _shape(4, 30, 4096, "f16", 1),      # whole accesses at an element's alignment
    _shape(4, 30, 4096, "f32", 3),
]
# Accesses of 8, 4 and 2 bytes: one slice per channel (the comparison blocks)
# on each rung and past it, and slices that exchange sums (the backward).
NARROW_BLOCKS = [
    _shape(9, 300, 196, "f16"), _shape(64, 300, 100, "f16"), _shape(64, 300, 196, "bf16"),
    _shape(150, 300, 196, "f16"),                                            # 8 bytes, past 16 accesses
    _shape(5, 300, 50, "f16"), _shape(250, 300, 50, "bf16"),                 # 4
    _shape(20, 300, 49, "f16"), _shape(40, 300, 49, "f16"), _shape(60, 300, 49, "bf16"),
    _shape(130, 300, 49, "f16"),                                             # 2, past 16 accesses
    _shape(30, 300, 30, "f32"), _shape(100, 300, 98, "f32"),                 # 8
    _shape(20, 300, 31, "f32"), _shape(100, 300, 31, "f32"),                 # 4
]
NARROW_EXCHANGE = [_shape(3000, 20, 52, "f16"), _shape(3000, 20, 50, "f16"), _shape(3000, 20, 49, "bf16"),
                   _shape(2600, 20, 30, "f32"), _shape(2600, 20, 31, "f32")]
# Channels cut into P slices (few, many, the most) that exchange sums.
EXCHANGE = [
    _shape(4, 40, 40000, "f16"),        # 12 slices
    _shape(2, 90, 66000, "f16"),        # 5
    _shape(3, 4, 524289, "f16"),        # 64, a tail
    _shape(2, 200, 25001, "bf16"),      # 2
    _shape(6, 20, 50176, "f32"),        # 25
]
CHECKS = [parity.test_random_shape_parity, parity.test_random_shape_backward_ii,
          parity.test_random_shape_standard_block, parity.test_random_shape_checkpointing]
ID = lambda v: (v if isinstance(v, str) else v.id if isinstance(v, parity.Shape) else  # noqa: E731
                v.__name__.replace("test_random_shape_", ""))


FORWARDS = ["forward_train", "std_forward", "ckpt_forward"]
BACKWARDS = ["backward", "std_backward", "ckpt_backward"]
BLOCKS = FORWARDS[1:] + BACKWARDS[1:]


# (Plans are those of aligned tensors.  (100, 300, 71): InPlace-ABN's own
# passes are channel-resident.)
@pytest.mark.parametrize("shapes, ops", [
    (TAILS + [s for s in SMALL if not s.offset and s.N != 100] + EXCHANGE + RUNGS, FORWARDS + BACKWARDS),
    ([s for s in SMALL if s.N == 100] + NARROW_BLOCKS, BLOCKS),
    (NARROW_EXCHANGE, BACKWARDS)], ids=["all", "blocks", "backwards"])
def test_takes_the_slices(shapes, ops):
    for s in shapes:
        for op in ops:
            p = iabn.iabn_plan(op, TORCH_DTYPES[s.dtype], s.N, s.C, s.HW)
            assert p["channel_resident"] == 0 and p["reg_accesses"] > 0, (s, op, p)
            narrow = s in NARROW_BLOCKS or s in NARROW_EXCHANGE
            assert (p["access_bytes"] < 16) == narrow, (s, op, p)
            exchange = s in EXCHANGE or s in NARROW_EXCHANGE
            assert (p["blocks"] > s.C) == exchange, (s, op, p)


@pytest.mark.parametrize("check", CHECKS, ids=ID)
@pytest.mark.parametrize("s", TAILS + SMALL + EXCHANGE + NARROW_EXCHANGE, ids=ID)
def test_slices(s, check):
    check(s)


@pytest.mark.parametrize("check", CHECKS[2:], ids=ID)
@pytest.mark.parametrize("s", NARROW_BLOCKS, ids=ID)
def test_narrow_blocks(s, check):
    check(s)


@pytest.mark.parametrize("check", CHECKS[:1] + CHECKS[2:3], ids=ID)
@pytest.mark.parametrize("s", RUNGS, ids=ID)
def test_rungs(s, check):
    check(s)


@pytest.mark.parametrize("s", TAILS + SMALL + EXCHANGE[2:4], ids=ID)
def test_inference(s):
    """The inference forward on the same rows (ragged ones by tiles too)."""
    inp = workloads.make_layer(s.N, s.C, s.HW, s.dtype, s.seed, gamma_sign=True)
    rm = np.linspace(-1.5, 1.5, s.C).astype(np.float32)
    rv = np.linspace(0.3, 4.0, s.C).astype(np.float32)
    buf, x = parity._placed(inp.x, s.dtype, s.offset, 5.5)
    iabn.iabn_forward_eval(x, *(torch.from_numpy(v).cuda() for v in (inp.gamma, inp.beta, rm, rv)),
                           1e-5, 0.01)
    torch.cuda.synchronize()
    ref = oracle.forward_eval(workloads.storage_to_f64(inp.x, s.dtype), inp.gamma, inp.beta, rm, rv,
                              parity.F32(1e-5), parity.F32(0.01))
    assert_close("z", to_f64(x), ref, s.dtype)
    assert parity._untouched(buf, s.offset, s.N * s.C * s.HW, 5.5)


# The recomputation's rules: few and many accesses per thread, few and many
# channels, against the general mapping's arithmetic (the forward's z).
@pytest.mark.parametrize("s", [_shape(8, 64, 4096, "f16"), _shape(2, 40, 20000, "bf16"),
                               _shape(2, 1030, 2048, "f16"), _shape(5, 1020, 1024, "f32")], ids=ID)
def test_recomputation(s):
    parity.test_random_shape_checkpointing(s)


@pytest.mark.parametrize("fn", [iabn.iabn_backward, iabn.iabn_backward_ii], ids=lambda f: f.__name__)
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("shape", [(2, 300, 9409), (3, 133, 9409), (2, 270, 5001)], ids=str)
def test_ragged_backward_sums_lose_no_small_terms(shape, dtype, fn):
    """Slices where the channel-resident kernels' elements one by one were
    before.  dz = (2^11, 2^-14, -2^11, 2^-14) over and over: an fp32 sum of two
    neighbours drops the small one, double holds every partial sum exactly, so
    dbeta and (xhat is 1) dgamma are the exact sum."""
    N, C, HW = shape
    dz = torch.tensor([2.0**11, 2.0**-14, -(2.0**11), 2.0**-14]).repeat(HW // 4 + 1)[:HW]
    dz[HW // 4 * 4:] = 0
    dz = dz.to(TORCH_DTYPES[dtype]).cuda().expand(N, C, HW).contiguous()
    u = torch.ones_like(dz)
    one, zero = torch.ones(C, device="cuda"), torch.zeros(C, device="cuda")
    dg, db = torch.empty(C, device="cuda"), torch.empty(C, device="cuda")
    plan = iabn.iabn_plan("backward", TORCH_DTYPES[dtype], N, C, HW)
    assert not plan["channel_resident"] and plan["reg_accesses"] > 0 and plan["access_bytes"] == 16, plan
    fn(u, dz, one, zero, one, dg, db)
    torch.cuda.synchronize()
    want = N * (HW // 4) * 2 * 2.0**-14
    assert bool((db == want).all()), (db[:4], want)
    assert bool((dg == want).all()), (dg[:4], want)


@pytest.mark.parametrize("shape", [(2, 300, 9409), (2, 40, 9409)], ids=str)
def test_alignment_moves_last_bits_only(shape):
    """Rows of 16-bit elements whose accesses start at a 16-byte boundary: the
    same bits at equal addresses modulo 16, else sums in another order.  A run
    of 8 fp32 terms is off by at most 8 * 2^-24 of the sum of their magnitudes,
    so two orders of a sum differ by at most U = 2^-20 of the sum of its terms'
    magnitudes: the mean and the variance of about the values' first and second
    absolute moments about a value of the channel (|x| < 6), dbeta and dgamma of
    the sums of |dy| and |dy xhat|.  What follows from them (z, dx) moves by
    that and a rounding to storage."""
    N, C, HW = shape
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x0, z0, dz0 = (torch.randn(shape, generator=g, device="cuda").half() for _ in range(3))
    one, zero = torch.ones(C, device="cuda"), torch.zeros(C, device="cuda")
    got = {}
    for off in (0, 8, 1, 3, 6):
        x, z, dz = (torch.empty(N * C * HW + 8, dtype=torch.half, device="cuda")[off:off + N * C * HW]
                    .view(shape).copy_(t) for t in (x0, z0, dz0))
        st = [torch.zeros(C, device="cuda") for _ in range(6)]
        iabn.iabn_forward_train(x, one, zero, *st[:4])
        iabn.iabn_backward(z, dz, one, zero, one, *st[4:])
        torch.cuda.synchronize()
        got[off] = [x, dz] + st
    for a, b in zip(got[0], got[8]):
        assert torch.equal(a, b)
    U, m = 2.0**-20, N * HW
    x, z, dz = (t.double() for t in (x0, z0, dz0))
    assert x.abs().max() < 6
    dy, w = torch.where(z < 0, 0.01 * dz, dz), torch.where(z < 0, z / 0.01, z)
    s_dy, s_dyw = dy.abs().sum((0, 2)), (dy * w).abs().sum((0, 2))
    stat = 37 * U  # (1 + 6^2) U
    bounds = [(12 * stat * torch.ones(C, device="cuda"), 2.0**-10),
              (U / m * (s_dy + w.abs().amax((0, 2)) * s_dyw), 2.0**-10)]
    bounds += [(stat, 0.0)] * 4 + [(U * s_dyw, 1e-6), (U * s_dy, 1e-6)]
    for off in (1, 3, 6):
        for i, (a, b, (bound, rel)) in enumerate(zip(got[0], got[off], bounds)):
            if i < 2:
                bound = bound.view(1, C, 1)
            a, b = a.double(), b.double()
            assert bool(((a - b).abs() <= bound + rel * a.abs() + 1e-7).all()), (off, i)


# Layers whose slices are abandoned: in 16-byte accesses, with edges, and in
# narrower ones (the backward only).
ABANDON_WIDE = [s for s in EXCHANGE if s.dtype in ("f16", "f32")]
ABANDON_NARROW = [s for s in NARROW_EXCHANGE if s.HW in (50, 31)]


@pytest.fixture
def abandoning(monkeypatch):
    """The binding on the library whose fp16 and fp32 kernels abandon the odd
    slices of a channel."""
    if not os.path.exists(iabn_build.ABANDON_LIB):
        iabn_build.build(abandon=True)
    lib = iabn.declare(ctypes.CDLL(iabn_build.ABANDON_LIB))
    monkeypatch.setattr(iabn, "_lib", lib)
    return lib


@pytest.mark.parametrize("check", CHECKS, ids=ID)
@pytest.mark.parametrize("s", ABANDON_WIDE + ABANDON_NARROW, ids=ID)
def test_abandoned_slices(s, check, abandoning):
    check(s)


def _one_op(op, L, ws):
    """One training entry point on copies of the layer's tensors; its outputs."""
    x, z, dz = L["x0"].clone(), L["z0"].clone(), L["dz0"].clone()
    v = {k: L[k].clone() for k in ("rm", "rv", "sm", "sv", "dg", "db")}
    a, kw = (L["g"], L["b"]), {"workspace": ws}
    stats = (v["rm"], v["rv"], v["sm"], v["sv"])
    if op == "forward_train":
        iabn.iabn_forward_train(x, *a, *stats, **kw)
    elif op == "std_forward":
        iabn.iabn_std_forward_train(x, z, *a, *stats, **kw)
    elif op == "ckpt_forward":
        iabn.iabn_ckpt_forward_train(x, z, *a, *stats, **kw)
    elif op == "backward":
        iabn.iabn_backward(z, dz, *a, v["sv"], v["dg"], v["db"], **kw)
    elif op == "std_backward":
        iabn.iabn_std_backward(x, z, dz, *a, v["sm"], v["sv"], v["dg"], v["db"], **kw)
    else:
        iabn.iabn_ckpt_backward(x, dz, *a, v["sv"], v["dg"], v["db"], **kw)
    torch.cuda.synchronize()
    return dict(v, x=x, z=z, dz=dz)


@pytest.mark.parametrize("s, op", [(s, op) for s in ABANDON_WIDE for op in FORWARDS + BACKWARDS] +
                         [(s, op) for s in ABANDON_NARROW for op in BACKWARDS], ids=ID)
def test_the_last_block_writes_abandoned_slices(s, op, abandoning, monkeypatch):
    """Bit for bit what the slices' own blocks write, and the flags in the
    workspace (behind the slots, 6 words twice for each slice) show that the
    last block did write them: every odd slice but its own."""
    plan = iabn.iabn_plan(op, TORCH_DTYPES[s.dtype], s.N, s.C, s.HW)
    slices = plan["blocks"]
    P = slices // s.C
    assert plan["reg_accesses"] > 0 and P > 3, plan
    L = test_gpu_streams._layer((s.N, s.C, s.HW), s.dtype, s.seed)
    L["z0"] = torch.randn_like(L["x0"])
    for k, v in dict(rm=0.0, sm=0.0, dg=0.0, db=0.0, rv=1.0, sv=1.0).items():
        L[k].fill_(v)
    say("abandoned %s %s" % (op, s.id))
    got = {}
    for name, lib in (("product", None), ("abandoning", abandoning)):
        with monkeypatch.context() as m:
            m.setattr(iabn, "_lib", lib)
            L["ws"].random_(0, 256)
            got[name] = _one_op(op, L, L["ws"])
    for k, v in got["product"].items():
        assert torch.equal(v, got["abandoning"][k]), k
    words = L["ws"][:slices * 16 * 8].view(torch.int64)
    marks = (words[slices * 12:slices * 13].view(s.C, P) == -1).sum(1)
    assert bool((marks >= P // 2 - 1).all()) and bool((marks <= P // 2).all()), marks


GRAPH = ((4, 40, 40000), "f16")


def test_graph_replay():
    test_gpu_graph.test_graph_replay_matches_eager(*GRAPH)


def test_graph_replay_ragged():
    test_gpu_graph.test_graph_replay_matches_eager((2, 100, 30003), "f16")


def test_graph_replay_abandoned(abandoning):
    test_gpu_graph.test_graph_replay_matches_eager(*GRAPH)


def _results(L):
    s = torch.cuda.current_stream()
    test_gpu_streams._run(L, s)
    torch.cuda.synchronize()
    return {k: L[k].clone() for k in ("x", "dz", "rm", "rv", "sm", "sv", "dg", "db")}


def test_workspace_content_does_not_matter():
    """Zeros, ones in every bit, random bytes, what other calls left: the same bits come out."""
    L = test_gpu_streams._layer((4, 40, 40000), "f16", 94)
    L["ws"].zero_()
    ref = _results(L)
    for what in ("ones", "random", "phases", "again"):
        say("workspace: %s" % what)
        if what == "ones":
            L["ws"].fill_(255)
        elif what == "random":
            L["ws"].random_(0, 256)
        elif what == "phases":
            iabn.iabn_forward_stats(L["x0"], L["ws"])
        got = _results(L)
        for k, v in ref.items():
            assert torch.equal(got[k], v), (what, k)


def test_concurrent_streams():
    """Layers on four streams at once (their blocks do not all fit the chip)
    give what they give one after the other."""
    layers = [test_gpu_streams._layer((4, 40, 40000), "f16", 95 + i) for i in range(3)]
    layers.append(test_gpu_streams._layer((2, 100, 30003), "f32", 99))
    ref = [_results(L) for L in layers]
    s0 = torch.cuda.current_stream()
    for rep in range(3):
        say("concurrent %d" % rep)
        streams = [torch.cuda.Stream() for _ in layers]
        for L, s in zip(layers, streams):
            s.wait_stream(s0)
            test_gpu_streams._run(L, s)
        for s in streams:
            s0.wait_stream(s)
        torch.cuda.synchronize()
        for L, r in zip(layers, ref):
            for k, v in r.items():
                assert torch.equal(L[k], v), k
