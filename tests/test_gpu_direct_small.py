"""GPU parity of the one-kernel float64 sums of small calls with the FP64
oracle, at the edges of its tiles (256 staged sources, 1 to 64 targets per
workgroup) and on both sides of the size rule, and of the kernels it stands in
for on the same inputs: a forced workgroup count keeps small calls on those.

Tolerance: FP64_TOL, the float64 bar of every direct sum (per pair ~4e-15 from
the Newton step, sums of at most 1e5 terms).
"""
import numpy as np
import pytest

import paper_1909_11085_amd as S
from oracle import oracle as O
from tests.gpu_util import FP64_TOL, assert_close, dev, host

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (255, 3), (256, 511), (257, 513), (1000, 1025), (40, 9001), (300, 33001), (20011, 65), (9001, 6660),
         (9001, 6670)]


def _case(seed, ns, nt):
    rng = np.random.default_rng(seed)
    y, x = rng.uniform(-3, 3, (3, ns)), rng.uniform(-3, 3, (3, nt))
    k = min(ns, nt, 5)
    x[:, :k] = y[:, :k]                                    # coincident points, any groups
    nv = rng.standard_normal((3, ns))
    return dict(y=y, x=x, f=rng.standard_normal((3, ns)), w=rng.uniform(0.1, 1.0, ns),
                n=nv / np.linalg.norm(nv, axis=0), gs=rng.integers(0, 4, ns).astype(np.int32),
                gt=rng.integers(0, 4, nt).astype(np.int32))


def _both(kernel, c, excl, **kw):
    kw.update(src_group=dev(c["gs"]), trg_group=dev(c["gt"]), exclude_same_group=excl)
    okw = dict(src_group=c["gs"], trg_group=c["gt"], exclude_same_group=excl)
    if kernel == "sl":
        return (S.sl(dev(c["y"]), dev(c["f"]), dev(c["w"]), dev(c["x"]), mu=1.3, **kw),
                O.sl(c["y"], c["f"], c["w"], c["x"], mu=1.3, **okw))
    return (S.dl(dev(c["y"]), dev(c["f"]), dev(c["w"]), dev(c["n"]), dev(c["x"]), **kw),
            O.dl(c["y"], c["f"], c["w"], c["n"], c["x"], **okw))


@pytest.mark.parametrize("kernel", ["sl", "dl"])
@pytest.mark.parametrize("excl", [True, False])
@pytest.mark.parametrize("sizes", SIZES)
@pytest.mark.parametrize("grid", [0, 768])
def test_sizes_match_oracle(kernel, excl, sizes, grid):
    c = _case(sum(sizes), *sizes)
    S.set_grid_override(grid)
    try:
        got, ref = _both(kernel, c, excl)
    finally:
        S.set_grid_override(0)
    assert_close(host(got), ref, FP64_TOL, f"{kernel} {sizes} {excl} grid={grid}")


def test_accumulates_and_repeats():
    c = _case(3, 700, 900)
    base = np.random.default_rng(4).standard_normal((3, 900))
    out = dev(base.copy())
    got, ref = _both("sl", c, True, out=out, accumulate=True)
    assert got is out
    assert_close(host(out) - base, ref, FP64_TOL, "accumulate")
    a, b = host(_both("dl", c, True)[0]), host(_both("dl", c, True)[0])
    assert np.array_equal(a, b)
