"""Float64 direct sums whose workgroups take whole 256-source chunks: a range takes
its chunks spread over all sources.

Values: against the FP64 oracle, at numbers of chunks where a step through them can
go wrong (powers of two, primes, Fibonacci numbers, a last chunk with one source) and
ranges that begin and end anywhere in a target block (forced workgroup counts).
Tolerance: FP64_TOL, the float64 bar of every direct sum.

Time: check points lie among the sources of their own patch, where the sub-tiles that
need the exclusion rules follow each other.  A boundary product may take at most 1.2
times as long as the double layer of as many sources and targets that lie apart
(masked pairs, upsampling and extrapolation are about a tenth), each the best of
several runs.  With the sub-tiles in order one range of a target block had all of
those: 1.3 times.
"""
import numpy as np
import pytest
import torch

import paper_1909_11085_amd as S
from paper_1909_11085_amd import workloads as W
from oracle import oracle as O
from tests.gpu_util import FP64_TOL, assert_close, dev, device, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", ["sl", "dl"])
@pytest.mark.parametrize("chunks,last,nt,grid", [(16, 256, 900, 1), (17, 1, 2500, 2), (31, 200, 1025, 3),
                                                 (34, 64, 4000, 7), (55, 255, 100, 3), (64, 256, 3000, 11)])
def test_values_of_spread_chunks(kernel, chunks, last, nt, grid):
    rng = np.random.default_rng(chunks * 1000 + nt)
    ns = 256 * (chunks - 1) + last
    y, x = rng.uniform(-4, 4, (3, ns)), rng.uniform(-4, 4, (3, nt))
    k = min(nt, 40)
    x[:, :k] = y[:, -k:]                                    # coincident points
    sg, tg = (np.arange(ns) // 300).astype(np.int32), rng.integers(-1, ns // 300, nt).astype(np.int32)
    f, w = rng.standard_normal((3, ns)), rng.uniform(0.1, 1.0, ns)
    nv = rng.standard_normal((3, ns))
    nv /= np.linalg.norm(nv, axis=0)
    kw = dict(src_group=dev(sg), trg_group=dev(tg))
    okw = dict(src_group=sg, trg_group=tg, exclude_same_group=True)
    S.set_grid_override(grid)
    try:
        if kernel == "sl":
            got, ref = S.sl(dev(y), dev(f), dev(w), dev(x), **kw), O.sl(y, f, w, x, **okw)
        else:
            got, ref = S.dl(dev(y), dev(f), dev(w), dev(nv), dev(x), **kw), O.dl(y, f, w, nv, x, **okw)
    finally:
        S.set_grid_override(0)
    assert_close(host(got), ref, FP64_TOL, f"{kernel} {ns} x {nt} grid {grid}")


def _best_ms(call):
    call()
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(10):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


def test_check_points_do_not_wait_for_one_range():
    s = W.cube_sphere(1.0, m=2, q=16, axes=(1.0, 0.9, 0.8))
    rng = np.random.default_rng(3)
    X, phi = dev(s.pos), dev(rng.standard_normal((3, s.n)))
    near = _best_ms(lambda: S.bie_apply(X, phi, s.meta["nodes_1d"], s.meta["weights_1d"], eta=2, p=8))
    ns, nt = s.n * 16, s.n * 9
    nv = rng.standard_normal((3, ns))
    y, q, w = dev(rng.uniform(0, 1, (3, ns))), dev(rng.standard_normal((3, ns))), dev(rng.uniform(0.1, 1, ns))
    n, x = dev(nv / np.linalg.norm(nv, axis=0)), dev(rng.uniform(2, 3, (3, nt)))
    apart = _best_ms(lambda: S.dl(y, q, w, n, x))
    assert near < 1.2 * apart, f"check points {near:.2f} ms, apart {apart:.2f} ms"
