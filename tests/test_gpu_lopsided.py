"""Direct sums whose two sizes are far apart: a few probe points at very many
sources, a few sources at very many targets.

Values: against the FP64 oracle at the edges of the one-kernel path's rule (72
tiles of 256 sources; 1.2e8 pairs up to 5 tiles, 2.6e7 beyond) and of its last
tile.  Tolerance: FP64_TOL, the float64 bar of every direct sum (MIXED_TOL in mixed precision).

Workspace: partial sums are for sub-tiles that hold sources.

Times: a call's own choice of kernels may take at most 1.5 times as long as the
kernels that cut the sources over the whole chip (a forced workgroup count keeps
a call on those), each the best of several runs.  One workgroup per target
walking all sources took 8 times as long, padding every few sources to a full
tile twice.
"""
import ctypes

import numpy as np
import pytest
import torch

import paper_1909_11085_amd as S
from paper_1909_11085_amd import _capi as C
from oracle import oracle as O
from tests.gpu_util import FP64_TOL, MIXED_TOL, assert_close, dev, device, host

pytestmark = pytest.mark.gpu


def _case(seed, ns, nt):
    rng = np.random.default_rng(seed)
    y = np.sort(rng.uniform(-20, 20, (3, ns)), axis=1)      # in order along a line: boxes of 64 are small
    y[1:] += rng.uniform(-1, 1, (2, ns))
    x = rng.uniform(-3, 3, (3, nt))
    k = min(ns, nt, 5)
    x[:, :k] = y[:, :k]                                      # coincident points
    nv = rng.standard_normal((3, ns))
    return y, rng.standard_normal((3, ns)), rng.uniform(0.1, 1.0, ns), nv / np.linalg.norm(nv, axis=0), x


@pytest.mark.parametrize("kernel", ["sl", "dl"])
@pytest.mark.parametrize("ns,nt", [(18432, 3), (18433, 3), (200_000, 2), (1, 70_001), (63, 50_000), (257, 20_000),
                                   (1280, 20_500), (1281, 20_296), (1281, 20_297)])
def test_values_at_the_edges(kernel, ns, nt):
    y, f, w, nv, x = _case(ns + nt, ns, nt)
    if kernel == "sl":
        got, ref = S.sl(dev(y), dev(f), dev(w), dev(x)), O.sl(y, f, w, x)
    else:
        got, ref = S.dl(dev(y), dev(f), dev(w), dev(nv), dev(x)), O.dl(y, f, w, nv, x)
    assert_close(host(got), ref, FP64_TOL, f"{kernel} {ns} x {nt}")


def _best_ms(call):
    call()
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(10):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


@pytest.mark.parametrize("kernel", ["sl", "dl"])
@pytest.mark.parametrize("ns,nt", [(1_000_000, 1), (1_000_000, 16), (400_000, 64), (1, 1_000_000), (64, 400_000)])
def test_no_slower_than_the_split_sum(kernel, ns, nt):
    y, f, w, nv, x = (dev(a) for a in _case(3, ns, nt))
    out = torch.empty((3, nt), dtype=torch.float64, device=device())
    call = (lambda: S.sl(y, f, w, x, out=out)) if kernel == "sl" else (lambda: S.dl(y, f, w, nv, x, out=out))
    own = _best_ms(call)
    S.set_grid_override(768)
    try:
        split = _best_ms(call)
    finally:
        S.set_grid_override(0)
    print(f"{kernel} {ns} x {nt}: {own:.3f} ms, split {split:.3f} ms", flush=True)
    assert own <= 1.5 * split, (own, split)


@pytest.mark.parametrize("op", [C.OP_SL, C.OP_DL])
def test_no_partial_sums_of_padding(op):
    """Mixed sums: 64 sources are one sub-tile of 64, 256 are four, and both have one
    record array of 256; what is left of the workspace is partial sums."""
    size, opts, nt = ctypes.c_size_t(), C.Opts(C.MIXED, 0), 65_536
    bytes_of = []
    for ns in (64, 256):
        assert C.lib().stokes_workspace_size(S.context(device()), op, ns, nt, 0, 0, ctypes.byref(opts),
                                             ctypes.byref(size)) == C.OK
        bytes_of.append(size.value)
    assert bytes_of[0] <= 0.5 * bytes_of[1], bytes_of


@pytest.mark.parametrize("kernel", ["sl", "dl"])
@pytest.mark.parametrize("ns,nt", [(1, 3000), (64, 70_000), (65, 513), (193, 9000), (1537, 1025)])
def test_mixed_values(kernel, ns, nt):
    y, f, w, nv, x = _case(ns, ns, nt)
    g, h = np.zeros(ns, np.int32), np.full(1, 0.2)
    kw = dict(src_group=dev(g), exclude_same_group=False, precision="mixed", group_h=dev(h))
    if kernel == "sl":
        got, ref = S.sl(dev(y), dev(f), dev(w), dev(x), **kw), O.sl(y, f, w, x)
    else:
        got, ref = S.dl(dev(y), dev(f), dev(w), dev(nv), dev(x), **kw), O.dl(y, f, w, nv, x)
    assert_close(host(got), ref, MIXED_TOL, f"{kernel} {ns} x {nt}")


@pytest.mark.parametrize("ns,nt,timed", [(544, 120_001, True), (192, 200_001, True), (1536, 20_001, False),
                                         (1537, 20_001, False), (2176, 30_001, False)])
def test_near_pairs(ns, nt, timed):
    """Mixed sums, a spherical group of points among targets spread around it, with
    float64 pairs within half a spacing (some in most sub-tiles, one in a thousand of
    all pairs): values on both sides of the 24 sub-tiles up to which the near pass
    notes such pairs in its float32 loop, and well below that they may add a tenth
    to the call's time (taken source by source they added a fifth to a quarter)."""
    rng = np.random.default_rng(ns)
    v = rng.standard_normal((3, ns))
    y, f, w = 2.0 * v / np.linalg.norm(v, axis=0), rng.standard_normal((3, ns)), rng.uniform(0.1, 1.0, ns)
    x = rng.uniform(-3, 3, (3, nt))
    x[:, :10] = y[:, :10]
    args = [dev(a) for a in (y, f, w, x)]
    kw = dict(src_group=dev(np.zeros(ns, np.int32)), exclude_same_group=False, precision="mixed")
    out = torch.empty((3, nt), dtype=torch.float64, device=device())
    spacing = [dev(np.full(1, h)) for h in (1e-9, 0.3)]
    times = [_best_ms(lambda: S.sl(*args, group_h=h, out=out, **kw)) for h in spacing]
    print(f"{ns} x {nt}: {times[0]:.3f} ms without near pairs, {times[1]:.3f} ms with", flush=True)
    i = np.arange(0, nt, 37)
    i[:10] = np.arange(10)
    assert_close(host(out)[:, i], O.sl(y, f, w, x[:, i]), MIXED_TOL, "near")
    assert not timed or times[1] <= 1.1 * times[0], times
