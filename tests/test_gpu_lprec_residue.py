"""The angle convolution of the log-polar method by residues of the fine angle:
every column length, one to sixteen fine angles per angle, sectors that end
inside a group of rows, and the whole-column forms beside it, against the FP64
oracle."""
import math

import numpy as np
import pytest

from oracle import lprec as olp
from paper_2209_08450_amd import synth
from tests._util import assert_parity, note, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2209_08450_amd import tp as mod
    return mod


# (angles, rows, detector, spans, oversampling) -> points of a column, fine angles per angle
CASES = [
    ((400, 3, 300, 3, 1.0), 256, 8),
    ((350, 2, 150, 3, 2.0), 256, 8),
    ((200, 1, 200, 3, 0.25), 512, 2),
    ((520, 5, 120, 2, 1.0), 512, 4),
    ((900, 2, 100, 3, 1.0), 1024, 1),
    ((1100, 2, 90, 2, 2.0), 1024, 2),
    ((2100, 2, 60, 3, 1.0), 2048, 1),
    ((5600, 1, 48, 3, 1.0), 4096, 1),
    ((11600, 1, 40, 3, 1.0), 8192, 1),
    ((60, 2, 200, 3, 1.0), 64, 32),     # whole columns, kernel column built at the launch
    ((64, 1, 360, 3, 2.0), 64, 128),    # whole columns from the kernel table
]


@pytest.mark.parametrize("case", CASES)
def test_residue_convolution_matches_oracle(tp, case):
    import torch
    (na, rows, n, spans, os_), points, fine = case
    g = tp.lprec_grid(na, n, spans=spans, os=os_)
    assert (g["NA"] // g["M"], g["M"]) == (points, fine), g
    s = synth.ellipsoid_scan_np(seed=na + n, n_angles=na, n_rows=rows, n_det=n, center=0.5 * n - 0.8, n_dark=2,
                                n_flat=2, n_ellipsoids=8)
    plan = tp.Plan(0.2 + np.arange(na) * math.pi / na, n, s.center)
    note(f"lprec residue {case}")
    out = tp.lprec_fbp_chunk(plan, to_dev(s.proj), to_dev(s.dark), to_dev(s.flat), spans=spans, os=os_)
    torch.cuda.synchronize()
    want = olp.lprec_fbp(s.proj, s.dark, s.flat, 0.2, s.center, spans=spans, os=os_)
    assert_parity(to_host(out).astype(np.float64), want, "f32", label=f"lprec residue {case}")


# detector -> points of a padded row: through LDS below 1024, in registers from
# there; an axis near the detector's edge and an odd last pair
@pytest.mark.parametrize("n,points", [(255, 512), (257, 1024), (512, 1024), (513, 2048), (1500, 4096), (2100, 8192)])
def test_row_splines_match_oracle(tp, n, points):
    import torch
    na, rows, N = 90, 3, 40
    s = synth.ellipsoid_scan_np(seed=n, n_angles=na, n_rows=rows, n_det=n, center=0.5 * n + 2.7, n_dark=2, n_flat=2,
                                n_ellipsoids=8)
    plan = tp.Plan(np.arange(na) * math.pi / na, n, s.center, N)
    note(f"lprec row splines {n} columns, {points} points")
    out = tp.lprec_fbp_chunk(plan, to_dev(s.proj), to_dev(s.dark), to_dev(s.flat))
    torch.cuda.synchronize()
    want = olp.lprec_fbp(s.proj, s.dark, s.flat, 0.0, s.center, N)
    assert_parity(to_host(out).astype(np.float64), want, "f32", label=f"lprec row splines {n}")
