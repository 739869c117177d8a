"""Faint scans: the FP32 paths hold their rows and spectra to a precision
relative to the sample, so their error does not grow as absorption falls.  The
negative logarithm, whose FP32 argument near 1 has an absolute precision, is
taken from the library's own normalisation on both sides; what follows it is
compared with the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2209_08450_amd import synth
from tests._util import REL_L2, note, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2209_08450_amd import tp as mod
    return mod


def _scan(contrast, na, rows, n, center):
    """16-bit counts whose largest line integral is `contrast`."""
    s = synth.ellipsoid_scan_np(seed=7, n_angles=na, n_rows=rows, n_det=n, center=center, n_dark=1, n_flat=1,
                                n_ellipsoids=12)
    p = np.maximum(oracle.normalize(s.proj, s.dark, s.flat), 0.0)  # [rows][angles][columns]
    p *= contrast / p.max()
    dark = np.full((1, rows, n), 100, dtype=np.uint16)
    flat = (64000 + np.random.default_rng(1).integers(0, 1000, (1, rows, n))).astype(np.uint16)
    gain = flat.astype(np.float64) - dark
    proj = np.rint(dark + gain * np.exp(-p.transpose(1, 0, 2))).astype(np.uint16)
    return proj, dark, flat, s.angles


def _error(tp, path, contrast):
    na, rows, n, center = 100, 3, 160, 79.2
    proj, dark, flat, angles = _scan(contrast, na, rows, n, center)
    plan = tp.Plan(angles, n, center)
    P, D, F = to_dev(proj), to_dev(dark), to_dev(flat)
    p = to_host(tp.normalize(P, D, F)).astype(np.float64)
    if path == "fourier":
        got = tp.fourier_fbp_chunk(plan, P, D, F)
        y, off = oracle.filter_rows_padded(p)
        want = oracle.fourier_backproject(y, angles, center + off, n)
    else:
        got = tp.fbp_chunk(plan, P, D, F, "f32")
        want = oracle.backproject(oracle.filter_rows(p), angles, center, n)
    return rel_l2(to_host(got), want)


# A relative error is the same at every contrast; a factor 2 for what the
# coarser steps of the counts make of the image.
@pytest.mark.parametrize("contrast", [1e-2, 1e-3, 1e-4])
@pytest.mark.parametrize("path", ["fourier", "f32"])
def test_error_does_not_grow_as_absorption_falls(tp, path, contrast):
    note(f"faint scan {path} {contrast:g}")
    full, faint = _error(tp, path, 1.0), _error(tp, path, contrast)
    note(f"faint scan {path}: rel-L2 {full:.3e} at 1, {faint:.3e} at {contrast:g}")
    assert full < REL_L2["f32"]
    assert faint < 2.0 * full
