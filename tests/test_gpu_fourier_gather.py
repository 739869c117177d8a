"""The Fourier gather on the matrix cores: one to five groups of four pairs of
slices, tiles reached by few and by many angles, more grid points than
frequency samples, and both ends of the radius, against the FP64 oracle's
direct sum and against the same slices reconstructed alone."""
import numpy as np
import pytest

import oracle
from paper_2209_08450_amd import synth
from tests._util import assert_parity, note, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2209_08450_amd import tp as mod
    return mod


# (angles, rows, detector, slice side, half width).  Pairs: 1, 4, 5, 8, 9 and 17,
# that is 1, 2 and 4 groups of four per work-group and a second work-group.
# Angles: 1 and 3 (a block of four not filled), 128 / 129 (all tiles of 32 x 32
# points / the middle ones of 16 x 16), 400.  Slices wider than the detector:
# 2, 4 and 8 grid points per frequency sample.
SHAPES = [
    (1, 1, 40, 40, 6),
    (3, 8, 33, 33, 6),
    (128, 9, 48, 48, 6),
    (129, 16, 64, 64, 6),
    (400, 17, 40, 40, 6),
    (150, 34, 36, 36, 6),
    (140, 18, 32, 64, 6),
    (30, 5, 16, 64, 6),
    (60, 10, 16, 128, 8),
    (90, 3, 64, 64, 8),
]


@pytest.mark.parametrize("shape", SHAPES)
def test_gather_matches_oracle(tp, shape):
    import torch
    na, rows, n, N, hw = shape
    s = synth.ellipsoid_scan_np(seed=na + rows + n, n_angles=na, n_rows=rows, n_det=n, center=0.5 * n - 1.3, n_dark=2,
                                n_flat=2, n_ellipsoids=8)
    plan = tp.Plan(s.angles, n, s.center, N)
    note(f"fourier gather {shape}")
    run = lambda r: tp.fourier_fbp_chunk(plan, to_dev(s.proj[:, r].copy()), to_dev(s.dark[:, r].copy()),
                                         to_dev(s.flat[:, r].copy()), half_width=hw)
    out = run(slice(0, rows))
    torch.cuda.synchronize()
    got = to_host(out).astype(np.float64)
    want = oracle.fourier_fbp(s.proj, s.dark, s.flat, s.angles, s.center, N, kind="ramp")
    assert_parity(got, want, "f32", label=f"fourier gather {shape}")
    # a pair's sums are formed in the same order whatever travels beside it
    last = (rows - 1) // 2 * 2
    assert np.array_equal(to_host(run(slice(last, rows))), to_host(out)[last:])
