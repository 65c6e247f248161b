"""Direct sums whose two sizes are far apart: a few probe points at very many
sources, a few sources at very many targets.

Values: against the FP64 oracle at the edges of the one-kernel path's rule (72
tiles of 256 sources; 1.2e8 pairs up to 5 tiles, 2.6e7 beyond) and of its last
tile.  Tolerance: FP64_TOL, the float64 bar of every direct sum.

Times: a call's own choice of kernels may take at most 1.5 times as long as the
kernels that cut the sources over the whole chip (a forced workgroup count keeps
a call on those), each the best of several runs.  One workgroup per target
walking all sources took 8 times as long, padding every few sources to a full
tile twice.
"""
import numpy as np
import pytest
import torch

import paper_1909_11085_amd as S
from oracle import oracle as O
from tests.gpu_util import FP64_TOL, assert_close, dev, device, host

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
