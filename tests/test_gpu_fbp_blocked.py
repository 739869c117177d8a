"""The fused chunk's backprojection from blocked rows: edges of its tiles, of
its groups of slices and of its blocks of angles, against the FP64 oracle, and
results that do not depend on which of its forms a call takes."""
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


def _scan(na, rows, n, c):
    return synth.ellipsoid_scan_np(seed=na + rows + n, n_angles=na, n_rows=rows, n_det=n, center=c, n_dark=2, n_flat=2,
                                   n_ellipsoids=12)


# (angles, rows, detector, slice side, axis): 16-voxel tiles up to 22 tiles of
# 32 a side, 32-voxel tiles above; 16, 32 and 64 slices per work-group (rows up
# to 16, 32 and more); blocks of 4 (FP32) and 8 angles; slices whose rows are
# and are not whole groups of 4 voxels; taps on both detector edges
SHAPES = [
    (1, 1, 17, 16, 8.0),
    (3, 8, 40, 33, 19.5),
    (4, 9, 64, 64, 31.75),
    (8, 16, 100, 17, 50.0),
    (9, 17, 90, 97, 44.1),
    (13, 33, 50, 65, 3.0),       # axis near the detector's edge
    (5, 65, 31, 40, 15.0),
    (7, 3, 760, 736, 380.4),     # 23 x 23 tiles of 32: not a power of two
    (6, 20, 700, 741, 349.9),
    (5, 40, 1030, 1024, 515.0),  # 32 x 32 tiles
]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
def test_blocked_rows_match_oracle(tp, shape, storage):
    na, rows, n, N, c = shape
    s = _scan(na, rows, n, c)
    plan = tp.Plan(s.angles, n, c, N)
    note(f"fbp blocked {shape} {storage}")
    got = to_host(tp.fbp_chunk(plan, to_dev(s.proj), to_dev(s.dark), to_dev(s.flat), storage)).astype(np.float64)
    # first and last slices of the chunk and one between: every group of slices' ends
    z = sorted({0, rows // 2, rows - 1})
    want = oracle.fbp(s.proj[:, z], s.dark[:, z], s.flat[:, z], s.angles, c, N=N)
    assert_parity(got[z], want, storage, label=f"blocked {shape}")


@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("N", [70, 745])
def test_blocked_rows_do_not_depend_on_the_chunk(tp, storage, N):
    # 70 rows in one call (64 slices per work-group), 24 (32) and 5 (16): the
    # rows they share are bitwise equal, the chunk a strided view of the scan
    import torch
    s = _scan(11, 70, 96, 47.0)
    plan = tp.Plan(s.angles, 96, 47.0, N)
    P, D, F = to_dev(s.proj), to_dev(s.dark), to_dev(s.flat)
    note(f"fbp blocked chunks {storage} N={N}")
    whole = tp.fbp_chunk(plan, P, D, F, storage)
    for z0, z1 in ((3, 27), (65, 70)):
        part = tp.fbp_chunk(plan, P[:, z0:z1], D[:, z0:z1], F[:, z0:z1], storage)
        assert torch.equal(part, whole[z0:z1]), (storage, z0, z1)
    if storage == "f16":
        half = tp.fbp_chunk(plan, P[:, 3:27], D[:, 3:27], F[:, 3:27], storage, out_dtype="f16")
        assert torch.equal(half, whole[3:27].half())


def test_blocked_rows_store_through_any_view(tp):
    # slices written at an address that is a multiple of their type's size only
    import torch
    s = _scan(9, 10, 64, 32.0)
    plan = tp.Plan(s.angles, 64, 32.0)
    P, D, F = to_dev(s.proj), to_dev(s.dark), to_dev(s.flat)
    note("fbp blocked, odd output address")
    for out_dtype, dt in (("f32", torch.float32), ("f16", torch.float16)):
        want = tp.fbp_chunk(plan, P, D, F, "f16", out_dtype=out_dtype)
        buf = torch.zeros(10 * 64 * 64 + 1, dtype=dt, device="cuda")
        out = buf[1:].view(10, 64, 64)
        tp.fbp_chunk(plan, P, D, F, "f16", out=out, out_dtype=out_dtype)
        assert torch.equal(out, want)
        assert buf[0] == 0
