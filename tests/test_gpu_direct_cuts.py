"""GPU parity of the one-sided direct sums where a workgroup's range of work
begins inside a 256-source chunk, and where few target blocks share many
near-pass rows: targets scattered among clusters, so that most waves have
near-pass sub-tiles everywhere, at forced workgroup counts that cut the
(target block, 64-source sub-tile) units at other places.

Tolerances: the bars of every direct sum (FP64_TOL, MIXED_TOL).
"""
import numpy as np
import pytest

import paper_1909_11085_amd as S
from oracle import oracle as O
from tests.gpu_util import FP64_TOL, MIXED_TOL, assert_close, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", ["sl", "dl"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("ns,nt,grid", [(4101, 517, 3), (4101, 517, 41), (4101, 517, 2000), (1500, 5000, 77),
                                        (65, 2049, 1000), (700, 1, 1)])
def test_scattered_targets(kernel, precision, ns, nt, grid):
    rng = np.random.default_rng(ns + nt + grid)
    g = np.arange(ns) // 150                              # clusters in source order
    c = rng.uniform(-4, 4, (3, g.max() + 1))
    y = c[:, g] + 0.5 * rng.standard_normal((3, ns))
    x = rng.uniform(-5, 5, (3, nt))
    x[:, : nt // 3] = y[:, rng.integers(0, ns, nt // 3)] + 0.02 * rng.standard_normal((3, nt // 3))
    x[:, 0] = y[:, -1]                                    # one coincident pair
    tg = rng.integers(-1, g.max() + 1, nt).astype(np.int32)
    f, w = rng.standard_normal((3, ns)), rng.uniform(0.1, 1.0, ns)
    nv = rng.standard_normal((3, ns))
    nv /= np.linalg.norm(nv, axis=0)
    sg = g.astype(np.int32)
    kw = dict(src_group=dev(sg), trg_group=dev(tg), precision=precision, group_h=dev(np.full(g.max() + 1, 0.1)))
    okw = dict(src_group=sg, trg_group=tg, exclude_same_group=True)
    S.set_grid_override(grid)
    try:
        if kernel == "sl":
            got = S.sl(dev(y), dev(f), dev(w), dev(x), **kw)
        else:
            got = S.dl(dev(y), dev(f), dev(w), dev(nv), dev(x), **kw)
    finally:
        S.set_grid_override(0)
    ref = O.sl(y, f, w, x, **okw) if kernel == "sl" else O.dl(y, f, w, nv, x, **okw)
    assert_close(host(got), ref, FP64_TOL if precision == "fp64" else MIXED_TOL, f"{kernel} {precision} {grid}")


@pytest.mark.parametrize("ns,nt", [(450_001, 2047), (32_768, 32_700), (450_001, 2049)])
def test_long_double_layer(ns, nt):
    """Eight targets per lane (and four, where the last target block would be
    mostly padding): sampled targets, the block's edges among them."""
    rng = np.random.default_rng(ns + nt)
    sg = (np.arange(ns) // 1000).astype(np.int32)
    y, x = rng.uniform(-4, 4, (3, ns)), rng.uniform(-4, 4, (3, nt))
    y[0] += 0.1 * (sg % 7)
    tg = rng.integers(-1, sg[-1] + 1, nt).astype(np.int32)
    x[:, 5] = y[:, -1]
    x[:, nt - 1] = y[:, 0]
    f, w = rng.standard_normal((3, ns)), rng.uniform(0.1, 1.0, ns)
    nv = rng.standard_normal((3, ns))
    nv /= np.linalg.norm(nv, axis=0)
    got = S.dl(dev(y), dev(f), dev(w), dev(nv), dev(x), src_group=dev(sg), trg_group=dev(tg))
    i = np.unique(np.concatenate([[0, 5, 63, 64, 511, 512, 2046, nt - 1], rng.integers(0, nt, 56)]))
    ref = O.dl(y, f, w, nv, x[:, i], src_group=sg, trg_group=tg[i], exclude_same_group=True)
    assert_close(host(got)[:, i], ref, FP64_TOL, f"dl {ns} {nt}")
