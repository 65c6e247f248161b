"""Each-pair-once sums at the launch shapes' edges: two, four and six rows per
lane, weighted ranges at about two units per workgroup (the least that takes
weights) and ranges that begin in a row block's weighted units.  Sampled points
against the float64 oracle, at the bar of every direct sum."""
import numpy as np
import pytest

import paper_1909_11085_amd as S
from oracle import oracle as O
from tests.gpu_util import FP64_TOL, assert_close, dev, host
from tests.test_gpu_sym import _shared

pytestmark = pytest.mark.gpu


# with `grid` workgroups (0: the chip's own number)
@pytest.mark.parametrize("n,grid", [(8191, 0), (11_265, 0), (15_361, 0), (12_288, 0), (98_305, 0), (3072, 84), (3073, 85),
                                    (6144, 7), (9217, 2), (9217, 300), (5121, 1)])
@pytest.mark.parametrize("adjoint", [False, True])
def test_shapes(n, grid, adjoint):
    print(f"case sym shapes n={n} grid={grid} adjoint={adjoint}", flush=True)
    pos, f, w, g = _shared(n + grid, n)
    rng = np.random.default_rng(n)
    i = np.unique(np.concatenate([[0, 63, 64, n - 65, n - 1], rng.integers(0, n, 123)]))
    P, F, Wt, G = dev(pos), dev(f), dev(w), dev(g)
    S.set_grid_override(grid)
    try:
        if not adjoint:
            got = host(S.sl(P, F, Wt, P, src_group=G, trg_group=G))[:, i]
        else:
            gv = rng.standard_normal((3, n))
            gf, gx = dev(np.full((3, n), np.nan)), dev(np.full((3, n), np.nan))
            S.sl_vjp(P, F, Wt, P, dev(gv), src_group=G, trg_group=G, grad_f=gf, grad_src=gx, grad_trg=gx)
            gf, gx = host(gf)[:, i], host(gx)[:, i]
    finally:
        S.set_grid_override(0)
    kw = dict(exclude_same_group=True)
    if not adjoint:
        assert_close(got, O.sl(pos, f, w, pos[:, i], src_group=g, trg_group=g[i], **kw), FP64_TOL, "velocity")
        return
    _, _, rt = O.sl_vjp(pos, f, w, pos[:, i], gv[:, i], src_group=g, trg_group=g[i], want=("trg",), **kw)
    rf, rs, _ = O.sl_vjp(pos[:, i], f[:, i], w[i], pos, gv, src_group=g[i], trg_group=g, want=("f", "src"), **kw)
    assert_close(gf, rf, FP64_TOL, "dL/df")
    assert_close(gx, rs + rt, FP64_TOL, "dL/dx")
