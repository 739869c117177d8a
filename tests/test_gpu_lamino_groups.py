"""The laminographic backprojection's groups of slices (2, 4 or 8 that share
their rows, by the sine of the tilt): both sides of each limit, slices that end
inside a block, and samples that are not finite, against the FP64 oracle."""
import math

import numpy as np
import pytest

import oracle
from tests._util import note, rel_l2, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2209_08450_amd import tp as mod
    return mod


def _case(seed, na, rows, n):
    q = np.random.default_rng(seed).standard_normal((na, rows, n)).astype(np.float32)
    return q, np.arange(na) * 2 * math.pi / na + 0.1


# sines 6/7 and 2/3 are the limits of 8 and 4 slices
@pytest.mark.parametrize("sine", [0.1, 0.66, 0.6667, 0.668, 0.8570, 0.8573, 0.93, 1.0])
@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
def test_groups_match_oracle(tp, sine, storage):
    import torch
    tilt = math.asin(sine)
    q, ang = _case(3, 22, 40, 50)
    N, Nz, cu, cv = 41, 21, 24.3, 19.6
    plan = tp.Plan(ang, 50, cu, N)
    qd = to_dev(q).to({"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[storage])
    note(f"lamino groups sine {sine} {storage}")
    got = to_host(tp.lamino_backproject(plan, qd, tilt, cv, Nz)).astype(np.float64)
    want = oracle.lamino_backproject(to_host(qd.float()).astype(np.float64), ang, cu, cv, tilt, N, Nz)
    assert rel_l2(got, want) < 1e-5
    assert np.max(np.abs(got - want)) < 1e-5 * np.max(np.abs(want))


@pytest.mark.parametrize("sine", [0.5, 0.75, 0.93])
@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("value", [math.inf, math.nan])
def test_a_sample_that_is_not_finite_reaches_its_own_taps_alone(tp, sine, storage, value):
    import torch
    tilt = math.asin(sine)
    na, rows, n, N, Nz, cu, cv = 9, 40, 50, 41, 13, 24.3, 19.6
    q, ang = _case(4, na, rows, n)
    a, r, c = 5, 20, 26
    plan = tp.Plan(ang, n, cu, N)
    dt = torch.float16 if storage == "f16" else torch.float32
    note(f"lamino sample {value} sine {sine} {storage}")
    clean = to_host(tp.lamino_backproject(plan, to_dev(q).to(dt), tilt, cv, Nz)).astype(np.float64)
    q[a, r, c] = value
    got = to_host(tp.lamino_backproject(plan, to_dev(q).to(dt), tilt, cv, Nz)).astype(np.float64)
    z, y, x = np.meshgrid(np.arange(Nz) - Nz // 2, np.arange(N) - N // 2, np.arange(N) - N // 2, indexing="ij")
    u = x * math.cos(ang[a]) + y * math.sin(ang[a]) + cu
    v = (-x * math.sin(ang[a]) + y * math.cos(ang[a])) * math.cos(tilt) + z * math.sin(tilt) + cv
    du, dv = np.floor(u + 1e-3), np.floor(v + 1e-3)
    lu, lv = np.floor(u - 1e-3), np.floor(v - 1e-3)
    # voxels that read the sample whichever way their coordinates round, and those that may
    surely = np.isin(c - du, (0, 1)) & np.isin(c - lu, (0, 1)) & np.isin(r - dv, (0, 1)) & np.isin(r - lv, (0, 1))
    may = (np.isin(c - du, (0, 1)) | np.isin(c - lu, (0, 1))) & (np.isin(r - dv, (0, 1)) | np.isin(r - lv, (0, 1)))
    bad = ~np.isfinite(got)
    assert surely.any() and bad[surely].all() and not bad[~may].any()
    assert np.max(np.abs(got[~bad] - clean[~bad])) < 1e-5 * np.max(np.abs(clean))
