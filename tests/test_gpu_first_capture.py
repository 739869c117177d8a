"""After tp_prepare the very first call of a kernel may be a graph capture: every
form of the fused chunk's backprojection whose staged blocks need more than the
default 64 KiB of LDS (more than 32 slices, or more than 16 FP32 ones; 16- and
32-voxel tiles), and tp_backproject's tuned tiling.  In a fresh process, where
no kernel has run; replays, with eager work between them, equal the eager call."""
import os
import subprocess
import sys

import pytest

from tests._util import note

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_SCRIPT = r"""
import sys
import numpy as np
import torch
sys.path.insert(0, sys.argv[1])
from paper_2209_08450_amd import synth, tp
from tests._util import to_dev


def captured(fn):
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=torch.cuda.Stream(), capture_error_mode="thread_local"):
        fn()
    return g


def check(label, g, out, eager, between):
    torch.cuda.synchronize()
    for rep in range(3):
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager), (label, rep)
        between()
        torch.cuda.synchronize()
    print("ok", label, flush=True)


na, rows, n = 24, 40, 64
s = synth.ellipsoid_scan_np(seed=12, n_angles=na, n_rows=rows, n_det=n, center=31.6, n_dark=2, n_flat=2)
P, D, F = to_dev(s.proj), to_dev(s.dark), to_dev(s.flat)
q = to_dev(np.random.default_rng(2).standard_normal((rows, na, n)).astype(np.float32)).half()
for N in (96, 740):
    plan = tp.Plan(s.angles, n, s.center, N)
    for storage, out_dtype, dt in (("f16", "f32", torch.float32), ("f16", "f16", torch.float16),
                                   ("bf16", "f32", torch.float32), ("f32", "f32", torch.float32)):
        print("case", N, storage, out_dtype, flush=True)
        plan.prepare("parzen", storage)
        out = torch.empty((rows, N, N), device="cuda", dtype=dt)
        ws = torch.empty(plan.fbp_workspace_bytes(rows, storage), dtype=torch.uint8, device="cuda")
        g = captured(lambda: tp.fbp_chunk(plan, P, D, F, storage, out=out, workspace=ws, kind="parzen",
                                          out_dtype=out_dtype))
        eager = tp.fbp_chunk(plan, P, D, F, storage, kind="parzen", out_dtype=out_dtype)
        check((N, storage, out_dtype), g, out, eager, lambda: tp.fbp_chunk(plan, P, D, F, storage, kind="shepp"))
    print("case", N, "tp_backproject", flush=True)
    plan.set_tuning("f16", 16, 32)  # 120.5 KiB staged
    plan.prepare("ramp", "f16")
    out = torch.empty((rows, N, N), device="cuda")
    g = captured(lambda: tp.backproject(plan, q, out=out))
    check((N, "tp_backproject"), g, out, tp.backproject(plan, q), lambda: tp.filter(q.float()))
    plan.close()
print("captures ok", flush=True)
"""


def test_first_calls_are_captures():
    note("first calls captured, in a child process")
    r = subprocess.run([sys.executable, "-c", _SCRIPT, ROOT], capture_output=True, text=True, timeout=100, cwd=ROOT)
    print(r.stdout[-3000:], r.stderr[-2000:], flush=True)
    assert r.returncode == 0
    assert "captures ok" in r.stdout
