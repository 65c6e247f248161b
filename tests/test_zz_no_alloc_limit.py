"""The allocation-free single-layer entry point near its limit in mixed precision
(about 300,000 points a side): bitwise the values of stokes_sl_eval with pair
symmetry off, and a sample of targets against the FP64 oracle (MIXED_TOL), where
that call's own scratch is more than the 64 MiB that sizes are accepted by.

stokes_sl_eval itself has no step there: with few targets the sizes just within
the limit (about 1,100,000 sources at 100 targets) take at most 1.15 times as long
as those just beyond, each the best of several runs.  Kept to 64 MiB it had two
thirds of the workgroups and 4 near-pass rows for 64.
"""
import numpy as np
import pytest
import torch

import paper_1909_11085_amd as S
from oracle import oracle as O
from paper_1909_11085_amd import _capi as C
from tests.gpu_util import MIXED_TOL, assert_close, dev, device, host
from tests.test_zz_no_alloc import _inputs, _noalloc, _reference, ctx  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [284_000, 290_000, 300_000])
def test_same_bits_near_the_limit(ctx, n):  # noqa: F811
    x = _inputs(41, n)
    assert C.lib().stokes_set_pair_symmetry(ctx, 0) == C.OK
    try:
        one, _ = _reference(ctx, x, C.MIXED)
    finally:
        assert C.lib().stokes_set_pair_symmetry(ctx, 1) == C.OK
    out = torch.full((3, n), np.nan, dtype=torch.float64, device=device())
    assert _noalloc(ctx, x, C.MIXED, out) == C.OK, C.lib().stokes_last_error()
    got = host(out)
    i = np.arange(0, n, n // 97)
    h = {k: host(x[k]) for k in ("pos", "f", "w", "grp")}
    ref = O.sl(h["pos"], h["f"], h["w"], h["pos"][:, i], mu=1.3, src_group=h["grp"], trg_group=h["grp"][i],
               exclude_same_group=True)
    assert_close(got[:, i], ref, MIXED_TOL, f"noalloc n={n}")
    assert np.array_equal(got, one)


def _best_ms(call):
    call()
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(15):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b))
    return best


def test_no_step_at_the_limit():
    rng = np.random.default_rng(6)
    x = dev(rng.uniform(-1, 1, (3, 100)))
    ms = {}
    for n in (1_070_000, 1_120_000):                      # 62.6 and 64.9 MiB by the measure of accepted sizes
        y = np.sort(rng.uniform(-100, 100, (3, n)), axis=1) + 5
        args = dev(y), dev(rng.standard_normal((3, n))), dev(rng.uniform(0.1, 1, n)), x
        ms[n] = _best_ms(lambda: S.sl(*args, precision="mixed"))
    assert ms[1_070_000] < 1.15 * ms[1_120_000], ms
