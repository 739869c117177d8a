"""The work whose time counts: one pass each of what programs ask of this library.

Every path that turns detector rows into slices, the differentiable projector
pair, the laminographic backprojector and the two row-wise steps, through the
public calls of ``paper_2209_08450_amd.tp`` and ``.autograd``, over the sizes
the repository's tests, benchmark and pipeline use and ragged ones between.
"""
import math

import numpy as np
import torch

from paper_2209_08450_amd import autograd, synth, tp

DEVICE = "cuda:0"


def _case(path, **kw):
    c = {"path": path, "rows": 1, "angles": 1, "det": 1, "vox": 0, "offset": 0.0, "storage": "f32", "window": "ramp",
         "out": "f32", "tilt": 0.0, "det_rows": 0}
    c.update(kw)
    c["vox"] = c["vox"] or c["det"]
    return c


def listed():
    return [
        # the 16-slice scan of the smoke check and the accuracy tests: launches and latency
        _case("fbp", name="scan_16_slices_f32", rows=16, angles=180, det=256),
        # one slice while a sample is aligned: the smallest useful call at a detector's full width
        _case("fbp", name="preview_1_slice_f32", rows=1, angles=900, det=1024, offset=3.25),
        # the 2048-cubed scan in chunks, rows stored in each precision
        _case("fbp", name="chunk_f16", rows=128, angles=2048, det=2048, storage="f16"),
        _case("fbp", name="chunk_f32", rows=32, angles=2048, det=2048),
        # nothing a power of two: axis off centre, slices narrower than the detector, smooth window
        _case("fbp", name="chunk_bf16_ragged", rows=37, angles=1201, det=1501, vox=1400, offset=-11.3, storage="bf16",
              window="parzen"),
        # the pipeline's smallest chunk of the 3000 x 2048 x 4096 scan, 16-bit slices for storage
        _case("fbp", name="chunk_f16_slices_wide", rows=32, angles=3000, det=4096, storage="f16", out="f16"),
        # the Fourier-domain method: a chunk of the 2048-cubed scan, and a ragged few rows
        _case("fourier", name="fourier_chunk", rows=64, angles=2048, det=2048),
        _case("fourier", name="fourier_ragged_f16_slices", rows=9, angles=721, det=900, offset=5.7, window="parzen",
              out="f16"),
        # the log-polar method: half a pipeline chunk of the 2048-cubed scan
        _case("lprec", name="lprec_chunk", rows=16, angles=2048, det=2048),
        # one gradient of the least-squares loss (forward and backward) as the iterative solver takes it
        _case("gradient", name="least_squares_gradient", rows=64, angles=900, det=1024),
        # a laminographic slab from 16-bit projections of a full turn
        _case("lamino", name="lamino_slab_f16", rows=64, angles=512, det=1024, det_rows=1024, storage="f16", tilt=1.1),
        # sinogram and filtered rows kept apart, as a program with steps of its own between them does
        _case("lines", name="normalize_then_filter", rows=48, angles=1800, det=1920, window="shepp", storage="f16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["fbp", "fbp", "fbp", "fourier", "lprec", "gradient", "lamino", "lines"])
    window = rng.choice(["ramp", "shepp", "parzen"])
    if path == "fbp":
        det, angles, rows = _log_int(rng, 180, 2400), _log_int(rng, 120, 2400), _log_int(rng, 1, 130)
        vox = det if rng.random() < 0.5 else int(det * rng.uniform(0.7, 1.2))
        rows = max(1, min(rows, int(2.5e11 / (float(vox) * vox * angles))))
        storage = rng.choice(["f32", "f16", "bf16"])
        out = "f16" if storage == "f16" and rng.random() < 0.3 else "f32"
        return _case(path, rows=rows, angles=angles, det=det, vox=vox, offset=round(rng.uniform(-0.05, 0.05) * det, 2),
                     storage=storage, window=window, out=out)
    if path == "fourier":
        det, angles, rows = _log_int(rng, 128, 2048), _log_int(rng, 90, 2048), _log_int(rng, 1, 40)
        return _case(path, rows=rows, angles=angles, det=det, offset=round(rng.uniform(-0.05, 0.05) * det, 2),
                     window=window, out=rng.choice(["f32", "f32", "f16"]))
    if path == "lprec":
        det, rows = _log_int(rng, 200, 1500), _log_int(rng, 1, 12)
        angles = int(det * rng.uniform(0.7, 1.3))
        return _case(path, rows=rows, angles=angles, det=det, offset=round(rng.uniform(-0.02, 0.02) * det, 2),
                     window=window)
    if path == "gradient":
        det, angles, rows = _log_int(rng, 96, 800), _log_int(rng, 60, 900), _log_int(rng, 1, 48)
        return _case(path, rows=rows, angles=angles, det=det, offset=round(rng.uniform(-3.0, 3.0), 2))
    if path == "lamino":
        det, angles, rows = _log_int(rng, 128, 800), _log_int(rng, 60, 600), _log_int(rng, 4, 48)
        return _case(path, rows=rows, angles=angles, det=det, det_rows=int(det * rng.uniform(0.6, 1.0)),
                     offset=round(rng.uniform(-3.0, 3.0), 2), storage=rng.choice(["f16", "f32", "bf16"]),
                     tilt=round(rng.uniform(0.6, 1.5), 3))
    det, angles, rows = _log_int(rng, 200, 3000), _log_int(rng, 90, 1800), _log_int(rng, 1, 32)
    return _case(path, rows=rows, angles=angles, det=det, window=window, storage=rng.choice(["f32", "f16", "bf16"]))


# ---------------------------------------------------------------------------
# Inputs, from the seed alone
# ---------------------------------------------------------------------------
def _scan(case, seed):
    """12-bit counts of a random ellipsoid phantom, with dark and flat frames."""
    return synth.ellipsoid_scan_torch(int(seed), case["angles"], case["rows"], case["det"], DEVICE,
                                      center=case["det"] / 2 + case["offset"], n_ellipsoids=24, n_dark=10, n_flat=10)


def _lamino_input(case, seed):
    g = torch.Generator(device=DEVICE).manual_seed(int(seed))
    q = torch.randn((case["angles"], case["det_rows"], case["det"]), generator=g, device=DEVICE)
    return q.to(tp.torch_dtype(tp.dtype_code(case["storage"])))


def _lamino_angles(case):
    return np.arange(case["angles"]) * (2.0 * math.pi / case["angles"])


def _gradient_input(case, seed):
    y, angles, _ = synth.ls_problem_torch(int(seed), case["rows"], case["det"], case["angles"], DEVICE, n_ellipsoids=24)
    g = torch.Generator(device=DEVICE).manual_seed(int(seed) + 1)
    x = torch.rand((case["rows"], case["vox"], case["vox"]), generator=g, device=DEVICE)  # an iterate of the solver
    return x, y, angles


def prepare(case, seed):
    path = case["path"]
    s = {"case": case}
    if path == "gradient":
        x, y, angles = _gradient_input(case, seed)
        s.update(x=x.requires_grad_(True), y=y,
                 plan=tp.Plan(angles, case["det"], case["det"] / 2 + case["offset"], case["vox"]))
        return s
    if path == "lamino":
        s["q"] = _lamino_input(case, seed)
        s["plan"] = tp.Plan(_lamino_angles(case), case["det"], (case["det"] - 1) / 2 + case["offset"], case["vox"])
        s["center_v"] = (case["det_rows"] - 1) / 2
        s["slices"] = 2 * case["rows"]  # the slab is the volume's middle half
        tp.lamino_prepare(s["plan"], case["tilt"], s["center_v"], s["slices"])
        s["out"] = torch.empty((case["rows"], case["vox"], case["vox"]), dtype=torch.float32, device=DEVICE)
        return s
    d = _scan(case, seed)
    s.update(proj=d.proj, dark=d.dark, flat=d.flat)
    if path == "lines":
        tp.filter_prepare(tp.pad_len(case["det"]), case["window"])
        return s
    s["plan"] = plan = tp.Plan(d.angles, case["det"], d.center, case["vox"])
    dt = torch.float16 if case["out"] == "f16" else torch.float32
    s["out"] = torch.empty((case["rows"], case["vox"], case["vox"]), dtype=dt, device=DEVICE)
    if path == "fbp":
        plan.prepare(case["window"], case["storage"])
        need = plan.fbp_workspace_bytes(case["rows"], tp.dtype_code(case["storage"]))
    elif path == "fourier":
        plan.fourier_prepare(case["window"])
        need = plan.fourier_workspace_bytes(case["rows"])
    else:
        plan.lprec_prepare(case["window"])
        need = plan.lprec_workspace_bytes(case["rows"])
    s["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEVICE)
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def run(s):
    case = s["case"]
    path = case["path"]
    if path == "fbp":
        return tp.fbp_chunk(s["plan"], s["proj"], s["dark"], s["flat"], case["storage"], out=s["out"],
                            workspace=s["workspace"], kind=case["window"], out_dtype=case["out"])
    if path == "fourier":
        return tp.fourier_fbp_chunk(s["plan"], s["proj"], s["dark"], s["flat"], out=s["out"], workspace=s["workspace"],
                                    kind=case["window"], out_dtype=case["out"])
    if path == "lprec":
        return tp.lprec_fbp_chunk(s["plan"], s["proj"], s["dark"], s["flat"], out=s["out"], workspace=s["workspace"],
                                  kind=case["window"])
    if path == "gradient":
        r = autograd.radon(s["x"], s["plan"]) - s["y"]
        (g,) = torch.autograd.grad((r * r).sum(), s["x"])
        return {"residual": r.detach(), "gradient": g}
    if path == "lamino":
        return tp.lamino_backproject(s["plan"], s["q"], case["tilt"], s["center_v"], s["slices"],
                                     z0=case["rows"] // 2, nz=case["rows"], out=s["out"])
    sino = tp.normalize(s["proj"], s["dark"], s["flat"])
    return {"sinogram": sino, "rows": tp.filter(sino, out_dtype=case["storage"], kind=case["window"])}


# ---------------------------------------------------------------------------
# What one pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    rows, na, n, N = case["rows"], case["angles"], case["det"], case["vox"]
    size = {"f32": 4, "f16": 2, "bf16": 2}
    L = tp.pad_len(n)
    raw = 2.0 * rows * na * n + 2.0 * 20 * rows * n
    fft = 5.0 * L * math.log2(L)  # one complex transform; two rows travel in it
    slices = float(rows) * N * N
    path = case["path"]
    if path == "fbp":  # two taps: four operations per voxel and angle
        return {"bytes": raw + slices * size[case["out"]], "flops": rows * na * fft + 4.0 * slices * na}
    if path == "fourier":  # every polar sample meets the grid points within 6 of it, then a 2-D transform
        M = max(L, tp.pad_len(N), 64)
        pairs = (rows + 1) // 2
        return {"bytes": raw + slices * size[case["out"]],
                "flops": pairs * (na * fft + 4.0 * math.pi * 36.0 * na * L + 10.0 * M * M * math.log2(M))}
    if path == "lprec":  # the transforms over log-radius and angle, and 36 taps per voxel and span
        g = tp.lprec_grid(na, N)
        pairs = (rows + 1) // 2
        col = 5.0 * g["NA"] * math.log2(g["NA"]) + 5.0 * (g["NA"] / g["M"]) * math.log2(g["NA"] / g["M"])
        line = 5.0 * g["Ns"] * math.log2(g["Ns"])
        return {"bytes": raw + slices * 4,
                "flops": pairs * (na * (3 * fft + line) + g["spans"] * (g["Ns"] * col + g["rows"] * line)) +
                2.0 * 36 * g["spans"] * slices}
    if path == "gradient":
        return {"bytes": slices * 8 + 8.0 * rows * na * n, "flops": 8.0 * slices * na}
    if path == "lamino":  # four taps
        return {"bytes": float(size[case["storage"]]) * na * case["det_rows"] * n + slices * 4,
                "flops": 8.0 * slices * na}
    return {"bytes": raw + (4.0 + size[case["storage"]]) * rows * na * n, "flops": rows * na * fft}


# ---------------------------------------------------------------------------
# The same results in 64 bits, by plain torch and numpy
# ---------------------------------------------------------------------------
def _response(L, window):
    """DFT of the band-limited windowed ramp's taps over [-L/2, L/2)."""
    m = np.arange(L // 2 + 1, dtype=np.float64)
    if window == "ramp":
        h = np.where(m % 2 == 1, -1.0 / (math.pi * np.maximum(m, 1.0)) ** 2, 0.0)
        h[0] = 0.25
    elif window == "shepp":
        h = 2.0 / (math.pi ** 2 * (1.0 - 4.0 * m * m))
    else:
        # (1/2) int_0^1 x W(x) cos(pi m x) dx, pieces of degree 4: Gauss-Legendre on short panels
        panels = max(2, 2 * ((L // 2 + 3) // 4))
        t, wt = np.polynomial.legendre.leggauss(12)
        edges = np.linspace(0.0, 1.0, panels + 1)
        x = (0.5 * (edges[1:] + edges[:-1])[:, None] + 0.5 * np.diff(edges)[:, None] * t).reshape(-1)
        wx = (0.5 * np.diff(edges)[:, None] * wt).reshape(-1)
        f = np.where(x <= 0.5, 1 - 6 * x ** 2 + 6 * x ** 3, 2 * (1 - x) ** 3) * x * wx * 0.5
        xt = torch.from_numpy(x).to(DEVICE)
        ft = torch.from_numpy(f).to(DEVICE)
        h = torch.cat([torch.cos(torch.from_numpy(k).to(DEVICE)[:, None] * math.pi * xt) @ ft
                       for k in np.array_split(m, max(1, len(m) * len(x) // 50_000_000 + 1))]).cpu().numpy()
    full = np.zeros(L)
    full[:L // 2 + 1] = h
    full[L // 2 + 1:] = h[1:L // 2][::-1]
    return torch.from_numpy(np.fft.fft(full).real).to(DEVICE)


def _counts(t):
    return t.to(torch.float64)  # 12-bit counts: the sign bit is never set


def _sinogram(d):
    D = _counts(d.dark).mean(0)
    den = torch.clamp_min(_counts(d.flat).mean(0) - D, 1.0)
    out = torch.empty((d.proj.shape[1], d.proj.shape[0], d.proj.shape[2]), dtype=torch.float64, device=DEVICE)
    for z in range(out.shape[0]):
        out[z] = -torch.log(torch.clamp_min((_counts(d.proj[:, z]) - D[z]) / den[z], 1e-6))
    return out


def _padded_spectrum(p, window):
    n = p.shape[-1]
    L = tp.pad_len(n)
    off = (L - n) // 2
    u = torch.nn.functional.pad(p[None], (off, L - n - off), mode="replicate")[0]
    return torch.fft.fft(u) * _response(L, window), off, L


def _filtered(p, window):
    out = torch.empty_like(p)
    for z in range(p.shape[0]):
        Q, off, _ = _padded_spectrum(p[z], window)
        out[z] = torch.fft.ifft(Q).real[..., off:off + p.shape[-1]]
    return out


def _grid(N):
    c = torch.arange(N, device=DEVICE, dtype=torch.float64) - N // 2
    return c[None, :], c[:, None]


def _taps(theta, center, N, n):
    """Lower tap of every voxel in a row padded by one zero in front and two behind, and its weight."""
    x, y = _grid(N)
    s = x * math.cos(theta) + y * math.sin(theta) + center
    j = torch.floor(s)
    w = s - j
    j = j.to(torch.int64) + 1
    off = (j < 0) | (j > n)  # both taps off the detector
    w = torch.where(off, torch.zeros_like(w), w)
    return torch.where(off, torch.full_like(j, n + 1), j).reshape(-1), w.reshape(-1)


def _backprojected(q, angles, center, N, scale):
    rows, na, n = q.shape
    qp = torch.nn.functional.pad(q, (1, 2))
    acc = torch.zeros((rows, N * N), dtype=torch.float64, device=DEVICE)
    for a in range(na):
        j, w = _taps(float(angles[a]), center, N, n)
        line = qp[:, a]
        step = line[:, 1:] - line[:, :-1]
        for z in range(0, rows, 8):
            acc[z:z + 8] += line[z:z + 8].index_select(1, j)
            acc[z:z + 8].addcmul_(step[z:z + 8].index_select(1, j), w)
    return (acc * scale).reshape(rows, N, N)


def _projected(x, angles, center, n):
    """Scatter of both taps, as differences of running sums over the voxels in the order of their lower tap."""
    rows, N = x.shape[0], x.shape[1]
    flat = x.reshape(rows, -1)
    out = torch.empty((rows, len(angles), n), dtype=torch.float64, device=DEVICE)
    for a in range(len(angles)):
        j, w = _taps(float(angles[a]), center, N, n)
        order = torch.argsort(j)
        ends = torch.bincount(j, minlength=n + 2).cumsum(0)
        v, w = flat.index_select(1, order), w[order]
        lo = torch.nn.functional.pad(torch.cumsum(v * (1.0 - w), 1), (1, 0)).index_select(1, ends)
        hi = torch.nn.functional.pad(torch.cumsum(v * w, 1), (1, 0)).index_select(1, ends)
        # tap t of the padded row takes the lower taps at t and the upper ones at t - 1
        line = torch.diff(lo, dim=1, prepend=torch.zeros_like(lo[:, :1]))
        line[:, 1:] += torch.diff(hi, dim=1, prepend=torch.zeros_like(hi[:, :1]))[:, :-1]
        out[:, a] = line[:, 1:n + 1]
    return out


def _interpolant_sum(p, angles, center, N, window, scale):
    """Every voxel's sum over angles of its padded filtered row's trigonometric
    interpolant: the row 16 times upsampled by a zero-padded transform, then
    eight-point Lagrange interpolation (error below 3e-9 of the row)."""
    rows, up, acc = p.shape[0], 16, None
    x, y = _grid(N)
    acc = torch.zeros((rows, N * N), dtype=torch.float64, device=DEVICE)
    nodes = np.arange(-3, 5)
    for a in range(p.shape[1]):
        Q, off, L = _padded_spectrum(p[:, a], window)
        h = L // 2
        big = torch.zeros((rows, up * L), dtype=torch.complex128, device=DEVICE)
        big[:, :h] = Q[:, :h]
        big[:, -h + 1:] = Q[:, h + 1:]
        big[:, h] = 0.5 * Q[:, h]
        big[:, -h] = 0.5 * Q[:, h]
        fine = torch.fft.ifft(big).real * up
        s = (x * math.cos(float(angles[a])) + y * math.sin(float(angles[a])) + center + off) * up
        j = torch.floor(s)
        t = (s - j).reshape(-1)
        j = j.to(torch.int64).reshape(-1)
        for i, node in enumerate(nodes):
            w = torch.ones_like(t)
            for other in nodes:
                if other != node:
                    w = w * (t - float(other)) / float(node - other)
            acc.addcmul_(fine.index_select(1, (j + int(node)) % (up * L)), w)
    return (acc * scale).reshape(rows, N, N)


def _lamino_exact(case, q):
    N, n, rows, cv = case["vox"], case["det"], case["det_rows"], (case["det_rows"] - 1) / 2
    cu, phi = (n - 1) / 2 + case["offset"], case["tilt"]
    x, y = _grid(N)
    slices, z0 = 2 * case["rows"], case["rows"] // 2
    out = torch.zeros((case["rows"], N, N), dtype=torch.float64, device=DEVICE)
    for a, theta in enumerate(_lamino_angles(case)):
        c, sn = math.cos(theta), math.sin(theta)
        img = torch.nn.functional.pad(q[a].to(torch.float64), (1, 1, 1, 1)).reshape(-1)
        u = (x * c + y * sn + cu).clamp(-1.0, float(n))  # the frame of zeros takes what lies off the detector
        fu = torch.clamp(torch.floor(u), max=n - 1)
        wu = u - fu
        base = -x * sn * math.cos(phi) + y * c * math.cos(phi) + cv
        for k in range(case["rows"]):
            v = (base + (z0 + k - slices // 2) * math.sin(phi)).clamp(-1.0, float(rows))
            fv = torch.clamp(torch.floor(v), max=rows - 1)
            wv = v - fv
            i = ((fv + 1) * (n + 2) + fu + 1).to(torch.int64)
            lo = img[i] * (1 - wu) + img[i + 1] * wu
            hi = img[i + n + 2] * (1 - wu) + img[i + n + 3] * wu
            out[k] += lo * (1 - wv) + hi * wv
    return out * (math.pi / case["angles"])


def exact(case, seed):
    path, na, N = case["path"], case["angles"], case["vox"]
    updates = float(case["rows"]) * N * N * na
    if updates > {"fbp": 2.8e11, "fourier": 1.2e10, "lprec": 1.2e10, "gradient": 1e10, "lamino": 4e10, "lines": 1e13}[path]:
        return None
    if path == "gradient":
        x, y, angles = _gradient_input(case, seed)
        center = case["det"] / 2 + case["offset"]
        r = _projected(x.to(torch.float64), angles, center, case["det"]) - y.to(torch.float64)
        return {"residual": r, "gradient": _backprojected(r, angles, center, N, 2.0)}
    if path == "lamino":
        return _lamino_exact(case, _lamino_input(case, seed))
    d = _scan(case, seed)
    p = _sinogram(d)
    if path == "lines":
        return {"sinogram": p, "rows": _filtered(p, case["window"])}
    if path == "fbp":
        return _backprojected(_filtered(p, case["window"]), d.angles, d.center, N, math.pi / na)
    return _interpolant_sum(p, d.angles, d.center, N, case["window"], math.pi / na)
