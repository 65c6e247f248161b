"""The two-sided double-layer adjoint sweep at the edges of its launch shapes
(targets per lane, sub-tiles, groups of target blocks)."""
import numpy as np
import pytest
import torch

import paper_1909_11085_amd as S
from oracle import oracle as O
from tests.gpu_util import FP64_TOL, assert_close, dev, device, host
from tests.test_gpu_direct import _cloud

pytestmark = pytest.mark.gpu


# one, two, four and six targets per lane, each with a full and a barely begun
# last target block and source sub-tile
@pytest.mark.parametrize("sizes", [(64, 256), (65, 257), (16384, 512), (16129, 513), (16384, 1024), (65281, 1025),
                                   (32768, 1536), (65537, 3071)])
@pytest.mark.parametrize("side", [True, False])
def test_sweep_edges(sizes, side):
    print(f"case dl sweep {sizes} {side}", flush=True)
    c = _cloud(500 + sizes[1], *sizes)
    ns, nt = sizes
    g = np.random.default_rng(sizes[0]).standard_normal((3, nt))
    gp, gs, gt = (torch.full((3, n), np.nan, dtype=torch.float64, device=device()) for n in (ns, ns, nt))
    S.dl_vjp(dev(c["y"]), dev(c["f"]), dev(c["w"]), dev(c["n"]), dev(c["x"]), dev(g), src_group=dev(c["gs"]),
             trg_group=dev(c["gt"]), exclude_same_group=True, grad_phi=gp, grad_src=gs if side else None, grad_trg=gt)
    rp, rs, rt = O.dl_vjp(c["y"], c["f"], c["w"], c["n"], c["x"], g, src_group=c["gs"], trg_group=c["gt"],
                          exclude_same_group=True)
    assert_close(host(gp), rp, FP64_TOL, "dL/dphi")
    assert_close(host(gt), rt, FP64_TOL, "dL/dtrg")
    if side:
        assert_close(host(gs), rs, FP64_TOL, "dL/dsrc")


@pytest.mark.parametrize("accumulate", [False, True])
def test_sweep_groups_of_target_blocks(accumulate):
    """200,000 shared points: the sources' partials are taken in two groups of
    target blocks.  One array for both position gradients, against the
    one-sided passes (whose route does not depend on the size)."""
    print(f"case dl sweep groups {accumulate}", flush=True)
    n = 200_000
    rng = np.random.default_rng(7)
    y, phi, nrm, g = (dev(rng.standard_normal((3, n))) for _ in range(4))
    w = dev(rng.uniform(0.5, 1.0, n))
    base = dev(rng.standard_normal((3, n)) * 1e3)
    gp, gpos = (base.clone() if accumulate else torch.full_like(base, np.nan) for _ in range(2))
    S.dl_vjp(y, phi, w, nrm, y, g, grad_phi=gp, grad_src=gpos, grad_trg=gpos, accumulate=accumulate)
    rp, rs, rt = (torch.empty_like(base) for _ in range(3))
    S.dl_vjp(y, phi, w, nrm, y, g, grad_phi=rp)
    S.dl_vjp(y, phi, w, nrm, y, g, grad_src=rs)
    S.dl_vjp(y, phi, w, nrm, y, g, grad_trg=rt)
    off = base if accumulate else 0.0
    assert_close(host(gp - off), host(rp), FP64_TOL, "dL/dphi")
    assert_close(host(gpos - off), host(rs + rt), FP64_TOL, "combined dL/dx total")
