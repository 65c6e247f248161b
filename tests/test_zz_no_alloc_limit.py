"""The allocation-free single-layer entry point near its limit in mixed precision
(about 300,000 points a side): bitwise the values of stokes_sl_eval with pair
symmetry off, and a sample of targets against the FP64 oracle (MIXED_TOL), where
that call's own scratch would not fit the library's array with all workgroups.
"""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1909_11085_amd import _capi as C
from tests.gpu_util import MIXED_TOL, assert_close, device, host
from tests.test_zz_no_alloc import _inputs, _noalloc, _reference, ctx  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [284_000, 290_000, 300_000])
def test_same_bits_near_the_limit(ctx, n):  # noqa: F811
    x = _inputs(41, n)
    assert C.lib().stokes_set_pair_symmetry(ctx, 0) == C.OK
    try:
        one, ws_bytes = _reference(ctx, x, C.MIXED)
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
    assert ws_bytes <= C.NOALLOC_SCRATCH_BYTES
