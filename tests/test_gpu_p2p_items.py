"""Float64 leaf-to-leaf sums and adjoints at the edges of a work item: every
number of targets at which the lanes per target or the targets per lane change,
source streams that end around the staging capacity, lists that cross it in the
middle of a leaf, more target groups than an item tracks, and coincident points.
Against the float64 oracle at the bar of every direct sum."""
import numpy as np
import pytest

import paper_1909_11085_amd as S
from oracle import oracle as O
from tests.gpu_util import FP64_TOL, assert_close, dev, host
from tests.test_gpu_p2p_vjp import _gpu, _layout, _oracle

pytestmark = pytest.mark.gpu


def _items(groups):
    rng = np.random.default_rng(groups)
    nt = list(range(1, 18)) + [31, 32, 33, 47, 48, 49, 63, 64, 65, 96, 127, 128, 129, 0, 200]
    ns = rng.permutation([0, 1, 2, 15, 16, 17, 63, 64, 65, 66, 100, 127, 128, 129, 130, 191, 192, 193, 256, 300] +
                         list(rng.integers(1, 90, len(nt) - 20)))
    so, to = np.concatenate([[0], np.cumsum(ns)]), np.concatenate([[0], np.cumsum(nt)])
    lists = [rng.choice(len(nt), rng.integers(0, 9), replace=False) for _ in nt]
    lists[3] = np.zeros(0, dtype=np.int64)
    uo = np.concatenate([[0], np.cumsum([len(v) for v in lists])])
    ul = np.concatenate(lists)
    y, x = rng.uniform(-3, 3, (3, so[-1])), rng.uniform(-3, 3, (3, to[-1]))
    x[:, ::17] = y[:, rng.integers(0, so[-1], x[:, ::17].shape[1])]      # coincident with some source
    n = rng.standard_normal((3, so[-1]))
    return dict(y=y, x=x, f=rng.standard_normal(y.shape), w=rng.uniform(0.5, 1.0, so[-1]),
                n=n / np.linalg.norm(n, axis=0), gu=rng.standard_normal(x.shape),
                gs=rng.integers(0, groups, so[-1]).astype(np.int32), gt=rng.integers(0, groups, to[-1]).astype(np.int32),
                so=so.astype(np.int64), to=to.astype(np.int64), ofs=uo.astype(np.int64), ul=ul.astype(np.int32))


@pytest.mark.parametrize("groups", [1, 2, 40])
@pytest.mark.parametrize("excl", [True, False])
@pytest.mark.parametrize("kernel", ["sl", "dl"])
def test_item_edges(kernel, excl, groups):
    print(f"case p2p items {kernel} excl={excl} groups={groups}", flush=True)
    d = _items(groups)
    lay = (d["so"], d["to"], d["ofs"], d["ul"])
    got = S.p2p_leaf(_layout(d), dev(d["y"]), dev(d["f"]), dev(d["w"]), dev(d["x"]), kernel=kernel, nrm=dev(d["n"]),
                     src_group=dev(d["gs"]), trg_group=dev(d["gt"]), exclude_same_group=excl)
    ref = O.p2p(int(kernel == "dl"), d["y"], d["f"], d["w"], d["x"], *lay, nrm=d["n"], src_group=d["gs"],
                trg_group=d["gt"], exclude_same_group=excl)
    assert_close(host(got), ref, FP64_TOL, "sum")
    for name, a, b in zip("f src trg".split(), _gpu(d, 1.3, excl, kernel=kernel), _oracle(d, 1.3, excl, kernel=kernel)):
        assert_close(host(a), b, FP64_TOL, name)


@pytest.mark.parametrize("n_leaves", [7, 2048, 2049, 4096 * 2048, 4096 * 2048 + 1])
def test_many_leaves(n_leaves):
    """The work items' prefix sum over one workgroup, several, and more than add
    up the sums before them: a few full leaves among empty ones, every list
    naming them all, so the result is the direct sum."""
    rng = np.random.default_rng(n_leaves % 1009)
    full = np.unique(np.clip([0, 1, 2046, 2047, 2048, n_leaves // 2, n_leaves - 2, n_leaves - 1], 0, n_leaves - 1))
    size = np.zeros(n_leaves, dtype=np.int64)
    size[full] = rng.integers(1, 90, full.size)
    ofs = np.concatenate([[0], np.cumsum(size)]).astype(np.int64)
    lists = np.zeros(n_leaves, dtype=np.int64)
    lists[full] = full.size
    uo = np.concatenate([[0], np.cumsum(lists)]).astype(np.int64)
    ul = np.tile(full, full.size).astype(np.int32)
    n = int(ofs[-1])
    y, f, w = rng.uniform(-3, 3, (3, n)), rng.standard_normal((3, n)), rng.uniform(0.5, 1.0, n)
    Y = dev(y)
    got = S.p2p_leaf((dev(ofs), dev(ofs), dev(uo), dev(ul)), Y, dev(f), dev(w), Y)
    assert_close(host(got), O.sl(y, f, w, y), FP64_TOL, f"{n_leaves} leaves")
