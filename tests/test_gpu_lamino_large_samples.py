"""A large finite sample of a laminographic projection reaches its own taps
alone: every voxel that does not read it keeps its sum bit for bit, in each
size of the groups of slices that share their rows."""
import math

import numpy as np
import pytest

from tests._util import note, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2209_08450_amd import tp as mod
    return mod


# 2, 4 and 8 slices a group, and slices whole rows apart
@pytest.mark.parametrize("sine", [0.5, 0.75, 0.93, 1.0])
@pytest.mark.parametrize("storage,value", [("f32", 1e8), ("f32", -1e30), ("f32", "lowest"), ("bf16", 1e8),
                                           ("bf16", -1e30), ("bf16", "lowest"), ("f16", "lowest")])
def test_a_large_sample_reaches_its_own_taps_alone(tp, sine, storage, value):
    import torch
    dt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[storage]
    x = torch.finfo(dt).min if value == "lowest" else value
    tilt = math.asin(sine)
    na, rows, n, N, Nz, cu, cv = 9, 40, 50, 41, 21, 24.3, 19.6
    q = np.random.default_rng(4).standard_normal((na, rows, n)).astype(np.float32)
    ang = np.arange(na) * 2 * math.pi / na + 0.1
    a, r, c = 5, 20, 26
    plan = tp.Plan(ang, n, cu, N)
    note(f"lamino sample {x:g} sine {sine} {storage}")
    qd = to_dev(q).to(dt)
    qd[a, r, c] = 0.0
    clean = to_host(tp.lamino_backproject(plan, qd, tilt, cv, Nz))
    qd[a, r, c] = x
    got = to_host(tp.lamino_backproject(plan, qd, tilt, cv, Nz))
    z, y, xx = np.meshgrid(np.arange(Nz) - Nz // 2, np.arange(N) - N // 2, np.arange(N) - N // 2, indexing="ij")
    u = xx * math.cos(ang[a]) + y * math.sin(ang[a]) + cu
    v = (-xx * math.sin(ang[a]) + y * math.cos(ang[a])) * math.cos(tilt) + z * math.sin(tilt) + cv
    # FP32 coordinates below 64 round by less than 1e-5: taps that may be read
    near = lambda s, t: np.isin(t - np.floor(s + 1e-4), (0, 1)) | np.isin(t - np.floor(s - 1e-4), (0, 1))
    may = near(u, c) & near(v, r)
    assert may.any() and not np.array_equal(got[may], clean[may])
    assert np.array_equal(got[~may], clean[~may])
