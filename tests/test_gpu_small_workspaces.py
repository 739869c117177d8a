"""Workspaces just large enough for one pair of rows (one row) of plainly laid
out intermediates are accepted, and give the same slices bit for bit."""
import math

import numpy as np
import pytest

from paper_2209_08450_amd import synth
from tests._util import note, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2209_08450_amd import tp as mod
    return mod


def _up(x, m=256):
    return -(-x // m) * m


def _scan(na, rows, n):
    s = synth.ellipsoid_scan_np(seed=na + rows + n, n_angles=na, n_rows=rows, n_det=n, center=0.5 * n - 0.8, n_dark=2,
                                n_flat=2, n_ellipsoids=8)
    return s, to_dev(s.proj), to_dev(s.dark), to_dev(s.flat)


def _buffer(nbytes):
    import torch
    return torch.full((nbytes,), 0xff, dtype=torch.uint8, device="cuda")  # NaN in every type


# rows of the convolution in plain order, rounded up to 16; columns by residue
# (256 and 512 points) and whole (64)
@pytest.mark.parametrize("na,n", [(257, 150), (369, 120), (520, 120), (60, 100)])
def test_lprec_rows_to_sixteen(tp, na, n):
    import torch
    rows = 5
    s, P, D, F = _scan(na, rows, n)
    plan = tp.Plan(0.2 + np.arange(na) * math.pi / na, n, s.center)
    g = tp.lprec_grid(na, n)
    df = int(tp._normalize_ws(rows, n))
    a = max(8 * na * 2 * tp.pad_len(n), 8 * g["spans"] * _up(g["rows"], 16) * g["Ns"])
    b = max(8 * g["spans"] * g["Ns"] * g["n_span"], 8 * g["spans"] * g["rows"] * g["nj"])
    note(f"lprec workspace {na} x {n}: {g['rows']} rows")
    want = tp.lprec_fbp_chunk(plan, P, D, F)
    got = tp.lprec_fbp_chunk(plan, P, D, F, workspace=_buffer(df + _up(a) + _up(b)))
    assert torch.equal(got, want)
    assert bool(torch.isfinite(want).all())


# exactly the rows asked for: one narrower block below 8 (tiles of 16 and, at
# N = 740, of 32), above that the whole blocks that fit and the rest behind them
@pytest.mark.parametrize("rows", [1, 2, 5, 7, 9, 15, 37])
@pytest.mark.parametrize("N", [60, 740])
@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
def test_fbp_rows_without_whole_blocks(tp, rows, N, storage):
    import torch
    na, n = 13, 71
    s, P, D, F = _scan(na, rows, n)
    plan = tp.Plan(s.angles, n, s.center, N)
    df, size = int(tp._normalize_ws(rows, n)), 4 if storage == "f32" else 2
    need = df + _up(rows * na * n * size)
    note(f"fbp workspace {rows} rows N={N} {storage}")
    for out_dtype in ("f32", "f16") if storage == "f16" else ("f32",):
        want = tp.fbp_chunk(plan, P, D, F, storage, out_dtype=out_dtype)
        got = tp.fbp_chunk(plan, P, D, F, storage, workspace=_buffer(need), out_dtype=out_dtype)
        assert torch.equal(got, want), out_dtype
        assert bool(torch.isfinite(want.float()).all())
    with pytest.raises(tp.TpError, match="workspace"):
        tp.fbp_chunk(plan, P, D, F, storage, workspace=_buffer(need - 256))


# spectra of one pair or two in plain rows: tiles of 32 and, from 129 angles, of
# 16 grid points, one and two grid points per frequency sample, an odd last row,
# rows through LDS (64 and 128 points) and in registers (1024)
@pytest.mark.parametrize("na,rows,n,N", [(40, 1, 40, 40), (129, 5, 64, 64), (140, 4, 32, 64), (200, 3, 300, 300),
                                         (700, 2, 64, 64)])
@pytest.mark.parametrize("out_dtype", ["f32", "f16"])
def test_fourier_spectra_of_one_pair(tp, na, rows, n, N, out_dtype):
    import torch
    s, P, D, F = _scan(na, rows, n)
    plan = tp.Plan(s.angles, n, s.center, N)
    L = tp.pad_len(n)
    M = max(L, tp.pad_len(N), 64)
    df = int(tp._normalize_ws(rows, n))
    note(f"fourier workspace {na} x {rows} x {n}, N={N} {out_dtype}")
    want = tp.fourier_fbp_chunk(plan, P, D, F, out_dtype=out_dtype)
    assert bool(torch.isfinite(want.float()).all())
    for pairs in (1, 2):
        need = df + _up(pairs * max(8 * na * (L + 1), 8 * _up(N, 16) * M)) + _up(pairs * 8 * M * M)
        got = tp.fourier_fbp_chunk(plan, P, D, F, workspace=_buffer(need), out_dtype=out_dtype)
        assert torch.equal(got, want), pairs
        if pairs == 1:
            with pytest.raises(tp.TpError, match="workspace"):
                tp.fourier_fbp_chunk(plan, P, D, F, workspace=_buffer(need - 256), out_dtype=out_dtype)
