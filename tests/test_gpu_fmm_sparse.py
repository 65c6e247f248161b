"""GPU parity of the FMM's M2L on both sides of the rule that leaves nearly empty
levels to pair sums (fewer sources and targets than half the boxes of the level
above, at orders 4 and 5; than these at order 6), at the tile edges of the convolution with enough points for it, and
where the spectra take several batches of planes and of target octets, against
the oracle FMM.

Bars: those of the other FMM parity tests at these orders (operators from two SVD
codes; measured 1.0e-13 at order 3, below 1e-9 at 4, 5.5e-8 at 6).

Times: a tree with a point in every fourth octet as pair sums (points x points of
the surfaces, 294 of 456 at order 5 against 6, squared 0.42): order 5 within 0.45
of the order 6 sum, and order 6's double layer, whose leaves would be a
convolution, within 1.15 of its single layer.  As convolutions they took 0.56 and
1.4.
"""
import numpy as np
import pytest
import torch

import paper_1909_11085_amd as S
from oracle import fmm as F
from tests.gpu_util import dev, host, rel_l2

pytestmark = pytest.mark.gpu

TOL = {3: 1e-11, 4: 1e-9, 6: 1e-6}
_plans = {}


def _plan(order):
    if order not in _plans:
        _plans[order] = S.FMMPlan(order)
    return _plans[order]


def _points(rng, octets, per, depth):
    """`per` points in each of `octets` boxes of level depth - 1 (x-major from a corner), in two of its children."""
    n = 2 ** (depth - 1)
    i = np.arange(octets).repeat(per)
    cell = np.stack([i // (n * n), i // n % n, i % n])
    child = np.where(np.arange(octets * per) % 2, i % 8, (3 * i + 1) % 8)
    half = np.stack([child & 1, child >> 1 & 1, child >> 2])
    return -1.0 + (cell + 0.5 * half + rng.uniform(0.01, 0.49, (3, octets * per))) * (2.0 / n)


def _check(kernel, order, depth, src, trg, seed, zero=0):
    """The last `zero` sources have no strength, and as many of the last targets are not compared."""
    rng = np.random.default_rng(seed)
    n = src.shape[1]
    f, w, nrm = rng.standard_normal((3, n)), rng.uniform(0.5, 1.0, n), rng.standard_normal((3, n))
    nrm /= np.linalg.norm(nrm, axis=0)
    m, mt = n - zero, trg.shape[1] - zero
    f[:, m:] = 0.0
    cube = ((0.0, 0.0, 0.0), 1.0, depth)
    if kernel == "sl":
        got = S.fmm_sl(_plan(order), dev(src), dev(f), dev(w), dev(trg), *cube)
        ref = F.fmm_sl(src[:, :m], f[:, :m], w[:m], trg[:, :mt], np.zeros(3), 1.0, depth, order)
    else:
        got = S.fmm_dl(_plan(order), dev(src), dev(f), dev(w), dev(nrm), dev(trg), *cube)
        ref = F.fmm_dl(src[:, :m], f[:, :m], w[:m], nrm[:, :m], trg[:, :mt], np.zeros(3), 1.0, depth, order)
    e = rel_l2(host(got)[:, :mt], ref)
    assert e < TOL[order], e


@pytest.mark.parametrize("kernel", ["sl", "dl"])
@pytest.mark.parametrize("octets,per,depth", [(1, 300, 4), (15, 18, 4), (16, 18, 4), (17, 18, 4), (127, 17, 5),
                                              (128, 17, 5), (129, 17, 5)])
def test_octet_counts_with_enough_points(octets, per, depth, kernel):
    rng = np.random.default_rng(7 * octets + depth)
    trg = _points(rng, octets, per, depth)
    src = np.concatenate([_points(rng, octets + 3, per, depth), rng.uniform(-1, 1, (3, 60))], axis=1)
    _check(kernel, 3, depth, src, trg, octets)


@pytest.mark.parametrize("kernel", ["sl", "dl"])
@pytest.mark.parametrize("ns,nt", [(255, 255), (256, 200), (200, 256), (700, 1), (1, 700), (3, 3), (31, 32)])
def test_rule_edges(ns, nt, kernel):
    rng = np.random.default_rng(ns + nt)
    _check(kernel, 4, 4, rng.uniform(-1, 1, (3, ns)), rng.uniform(-1, 1, (3, nt)), 5)


@pytest.mark.parametrize("n", [63, 64])
def test_rule_edges_at_order_6(n):
    rng = np.random.default_rng(n)
    _check("dl", 6, 3, rng.uniform(-1, 1, (3, n)), rng.uniform(-1, 1, (3, n)), 6)


@pytest.mark.parametrize("kernel", ["sl", "dl"])
def test_batches_of_planes_and_targets(kernel):
    """262,144 octets at order 4: a plane a batch, two shares of the targets."""
    rng = np.random.default_rng(9)
    near = lambda n: -0.9 + 0.3 * rng.uniform(0, 1, (3, n))
    pad = 262_200
    src = np.concatenate([near(40), rng.uniform(0.5, 1, (3, 20)), rng.uniform(-1, 1, (3, pad))], axis=1)
    trg = np.concatenate([near(30), rng.uniform(0.4, 1, (3, 30)), rng.uniform(-1, 1, (3, pad))], axis=1)
    _check(kernel, 4, 7, src, trg, 10, zero=pad)


@pytest.mark.parametrize("pad", [3000, 60_000])
def test_exact_product_in_parts_and_whole(pad):
    """Order 6, double layer, depth 5: up to 16,384 leaves holding targets the exact pseudo-inverse product
    splits its sums, beyond it does not (60,000 points hold about 27,000); 4,096 points and more make the
    leaves a convolution."""
    rng = np.random.default_rng(12)
    near = lambda n: -0.7 + 0.4 * rng.uniform(0, 1, (3, n))
    src = np.concatenate([near(25), rng.uniform(0.5, 1, (3, 5)), rng.uniform(-1, 1, (3, pad + 1200))], axis=1)
    trg = np.concatenate([near(20), rng.uniform(0.4, 1, (3, 10)), rng.uniform(-1, 1, (3, pad + 1200))], axis=1)
    _check("dl", 6, 5, src, trg, 13, zero=pad + 1200)


def test_exact_product_has_no_rounding():
    """The same targets, one in every octet, alone (4,096 leaves, the exact product's sums split) and with others
    in 20,480 more leaves (not split): all upper levels and the leaves' check vectors are the same bits, so only
    the order of that product's sums differs.  What it leaves in float64 is 2^-21 of a plain product's rounding
    (which moves results by up to 1e-9) and one rounding of the densities: 1e-12 is a hundred times that."""
    rng = np.random.default_rng(14)
    n = 16
    cell = np.stack(np.meshgrid(*[np.arange(n)] * 3, indexing="ij")).reshape(3, -1)
    src = -1.0 + (cell + rng.uniform(0.01, 0.99, cell.shape)) * (2.0 / n)
    own = -1.0 + (cell + rng.uniform(0.01, 0.49, cell.shape)) * (2.0 / n)
    more = [own]
    for child in range(3, 8):
        half = 0.5 * np.array([child & 1, child >> 1 & 1, child >> 2])[:, None]
        more.append(-1.0 + (cell + half + 0.25) * (2.0 / n))
    f, w, nrm = rng.standard_normal(src.shape), rng.uniform(0.5, 1.0, src.shape[1]), rng.standard_normal(src.shape)
    nrm /= np.linalg.norm(nrm, axis=0)
    args = _plan(6), dev(src), dev(f), dev(w), dev(nrm)
    cube = ((0.0, 0.0, 0.0), 1.0, 5)
    split = host(S.fmm_dl(*args, dev(own), *cube))
    whole = host(S.fmm_dl(*args, dev(np.concatenate(more, axis=1)), *cube))[:, : own.shape[1]]
    e = rel_l2(split, whole)
    assert e < 1e-12, e


def _best_ms(call):
    call()
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


def test_sparse_trees_run_as_pair_sums():
    n, cube = 8192, ((0.0, 0.0, 0.0), 1.0, 6)
    rng = np.random.default_rng(11)
    src, trg, f, nrm = (dev(rng.uniform(-1, 1, (3, n))) for _ in range(4))
    w = dev(np.ones(n))
    sl6 = _best_ms(lambda: S.fmm_sl(_plan(6), src, f, w, trg, *cube))
    dl6 = _best_ms(lambda: S.fmm_dl(_plan(6), src, f, w, nrm, trg, *cube))
    dl5 = _best_ms(lambda: S.fmm_dl(_plan(5), src, f, w, nrm, trg, *cube))
    print(f"order 6: {sl6:.2f} ms, double layer {dl6:.2f}; order 5: {dl5:.2f}", flush=True)
    assert dl6 <= 1.15 * sl6 and dl5 <= 0.45 * sl6, (sl6, dl6, dl5)
