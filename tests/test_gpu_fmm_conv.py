"""GPU parity of the FMM's lattice-convolution M2L at the edges of its tiles:
octets (boxes of the level above the leaves) one short of, equal to and one
past a 16-column tile (few octets: the four waves of a workgroup share a tile)
and a 128-column workgroup (more than 512 targets: each wave has its own
columns), single and double layer, against the oracle FMM.

Order 3 keeps the oracle quick; the bar is the one of the other FMM parity
tests at that order (operators from two SVD codes, measured 1.0e-13).
"""
import numpy as np
import pytest

import paper_1909_11085_amd as S
from oracle import fmm as F
from tests.gpu_util import dev, host, rel_l2

pytestmark = pytest.mark.gpu

TOL = 1e-11


def _points_in_octets(rng, octets, per, depth):
    """`per` points in each of `octets` boxes of level depth - 1 (consecutive in x-major order from a corner)."""
    n = 2 ** (depth - 1)
    idx = np.arange(octets)
    cell = np.stack([idx // (n * n), idx // n % n, idx % n]).repeat(per, axis=1)
    return -1.0 + (cell + rng.uniform(0.01, 0.99, (3, octets * per))) * (2.0 / n)


@pytest.mark.parametrize("octets,per,depth", [(1, 1, 3), (15, 2, 4), (16, 2, 4), (17, 2, 4), (127, 5, 5), (128, 5, 5),
                                              (129, 5, 5)])
@pytest.mark.parametrize("kernel", ["sl", "dl"])
def test_octet_counts_match_oracle(octets, per, depth, kernel):
    rng = np.random.default_rng(7 * octets + depth)
    trg = _points_in_octets(rng, octets, per, depth)
    src = np.concatenate([_points_in_octets(rng, octets + 3, 1, depth), rng.uniform(-1, 1, (3, 150))], axis=1)
    n = src.shape[1]
    f, w = rng.standard_normal((3, n)), rng.uniform(0.5, 1.0, n)
    plan, cube = S.FMMPlan(3), ((0.0, 0.0, 0.0), 1.0, depth)
    if kernel == "sl":
        got = host(S.fmm_sl(plan, dev(src), dev(f), dev(w), dev(trg), *cube))
        ref = F.fmm_sl(src, f, w, trg, np.zeros(3), 1.0, depth, 3)
    else:
        nrm = rng.standard_normal((3, n))
        nrm /= np.linalg.norm(nrm, axis=0)
        got = host(S.fmm_dl(plan, dev(src), dev(f), dev(w), dev(nrm), dev(trg), *cube))
        ref = F.fmm_dl(src, f, w, nrm, trg, np.zeros(3), 1.0, depth, 3)
    assert rel_l2(got, ref) < TOL, rel_l2(got, ref)
