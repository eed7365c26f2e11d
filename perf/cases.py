"""The work that is measured: single calls as a reconstruction program makes them.

A case is one call (or one operator pair) through the package's public entry
points on device-resident data of one scan geometry:

* ``fbp``      filtered back-projection of a slab of sinograms (xct.fbp)
* ``batch``    the uneven batch: slabs of several sizes in one xct_fbp_batch call
* ``offset``   full-turn offset scan (xct.fbp_offset)
* ``front``    raw detector counts to filtered rows (xct_preprocess_filter)
* ``codes``    filtered rows to the stored volume's 16-bit CT-number codes
               (xct_backproject_u16)
* ``project``  the differentiable projector, forward and backward
* ``residual`` one least-squares iteration's operators: r = y - P x, P^T r

Inputs are line integrals of random ellipses with noise, in the storage type
of the case, on the device.  ``listed`` holds the sizes of the repository's
own workloads (a 256^2 slice up to the 16 x 8192^2 slab) and some that its
tests stand for; ``draw`` gives more of the same ranges.
"""

from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2505_13955_amd as xct

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "f16": 2, "bf16": 2}
CODE_WATER, CODE_MIN, CODE_MAX = 0.3, -1000.0, 4000.0  # CT-number range of the stored volume
FLOOR = 1.0                                            # counts
EXACT_UPDATES = 7e10                                   # some seconds of 64-bit gathers


def _scan(kind, n, angles, det, slices, **kw):
    c = {"kind": kind, "nx": n, "ny": n, "angles": angles, "det": det, "slices": slices,
         "center": (det - 1) / 2.0, "pixel": 1.0, "window": "ram_lak", "storage": "f32",
         "filtered": "f32", "sigma": 0.0, "overlap": 0.0}
    c.update(kw)
    return c


def listed():
    return [
        # one small slice: the quick look while a sample is aligned (latency)
        _scan("fbp", 256, 360, 367, 1, name="fbp_1x256"),
        # a preview of three slices of a cropped field whose axis was calibrated
        # to a fraction of a bin, odd sizes throughout
        _scan("fbp", 1001, 1201, 1425, 3, ny=903, center=703.37, window="shepp_logan", storage="bf16",
              name="fbp_3x1001_fractional_axis"),
        # the ordinary slab
        _scan("fbp", 2048, 1800, 2900, 64, window="shepp_logan", name="fbp_64x2048"),
        # the slab at the paper's resolution
        _scan("fbp", 8192, 6144, 8192, 16, window="hann", name="fbp_16x8192"),
        # reduced storage of scan and filtered rows
        _scan("fbp", 4096, 3072, 4096, 4, window="hann", storage="f16", filtered="f16", name="fbp_4x4096_f16"),
        # an angle count that no quarter turn maps onto itself
        _scan("fbp", 8192, 6143, 8192, 4, window="hann", name="fbp_4x8192_odd_angles"),
        # specimens of several sizes in one call
        _scan("batch", 2048, 2048, 2898, 4, storage="bf16", name="batch_uneven"),
        # an object wider than the detector, scanned over a full turn
        _scan("offset", 4096, 8192, 4096, 8, center=1024.0, overlap=1024.0, window="hann", name="offset_8x4096"),
        # raw counts of a slab of detector rows to filtered rows
        _scan("front", 2048, 1800, 2900, 32, window="hann", sigma=1.0, name="front_32x2900"),
        # the volume-storage end of the pipeline
        _scan("codes", 2048, 1800, 2900, 8, name="codes_8x2048"),
        # the differentiable pair at its benchmark size
        _scan("project", 1024, 1440, 1449, 32, name="project_32x1024"),
        # an iterative reconstruction of a single slice
        _scan("residual", 512, 720, 727, 1, name="residual_1x512"),
    ]


def draw(rng):
    kind = rng.choice(["fbp", "fbp", "fbp", "fbp", "batch", "offset", "front", "codes", "project", "residual"])
    top = {"project": 1400, "residual": 1000}.get(kind, 3200)
    n = int(round(math.exp(rng.uniform(math.log(120), math.log(top)))))
    square = rng.random() < 0.7
    if square and rng.random() < 0.7:
        n += n & 1
    angles = max(24, int(n * rng.uniform(0.6, 1.6)))
    if rng.random() < 0.6:
        angles += (-angles) % 4
    limit = 6e10 if kind in ("project", "residual") else 3e11
    most = max(1, min(32, int(limit / (float(n) * n * angles))))
    slices = int(round(math.exp(rng.uniform(0.0, math.log(most + 0.49)))))
    det = min(8192, int(math.ceil(math.sqrt(2.0) * n)) + rng.randint(1, 12)) if rng.random() < 0.7 else n + rng.randint(0, 9)
    c = _scan(kind, n, angles, det, max(1, slices), window=rng.choice(["ram_lak", "shepp_logan", "hann"]))
    if not square:
        c["ny"] = max(64, int(n * rng.uniform(0.6, 1.4)))
    where = rng.random()
    if where < 0.25:
        c["center"] += rng.randint(-8, 8) * 0.5
    elif where < 0.5:
        c["center"] += round(rng.uniform(-4.0, 4.0), 3)
    if rng.random() < 0.2:
        c["pixel"] = round(rng.uniform(0.7, 1.3), 3)
    if kind in ("fbp", "batch", "offset", "codes"):
        c["storage"] = rng.choice(["f32", "f32", "f16", "bf16"])
        c["filtered"] = rng.choice(["f32", "f32", "f32", "f16"]) if kind != "codes" else "f32"
    if kind == "front":
        c["sigma"] = rng.choice([0.0, 0.7, 1.0, 2.0])
    if kind == "offset":
        # the axis a quarter of the way along the detector, a full turn
        c["angles"] = max(32, angles + (-angles) % 4)
        c["det"] = n + rng.randint(0, 9)
        c["center"] = float(c["det"] // 4)
        c["overlap"] = float(max(2, int(c["center"] * rng.uniform(0.5, 1.0))))
    return c


# ---------------------------------------------------------------- scans

def _geometries(case):
    """(geometry, slices, overlap) of each slab of the case."""
    def geom(nx, ny, na, nd, center):
        turn = 2.0 * math.pi if case["overlap"] > 0 else math.pi
        return SimpleNamespace(n_angles=na, n_det=nd, nx=nx, ny=ny, det_pitch=1.0,
                               pixel_size=float(case["pixel"]), center=float(center),
                               angles=np.arange(na, dtype=np.float64) * (turn / na))
    base = geom(case["nx"], case["ny"], case["angles"], case["det"], case["center"])
    slabs = [(base, case["slices"], case["overlap"])]
    if case["kind"] == "batch":
        # the smaller specimens of the same call: half and a quarter of the size,
        # three and six times the slices
        for div, times, per in ((2, 3, 1440 / 2048), (4, 6, 720 / 2048)):
            nx, ny = max(48, case["nx"] // div), max(48, case["ny"] // div)
            nd = int(math.ceil(math.sqrt(2.0) * max(nx, ny))) + 1
            slabs.append((geom(nx, ny, max(16, int(case["angles"] * per)), nd, (nd - 1) / 2.0),
                          case["slices"] * times, 0.0))
    return slabs


def _updates(case):
    return sum(float(g.nx) * g.ny * g.n_angles * s for g, s, _ in _geometries(case))


def _ellipses(gen, n=8):
    """n ellipses inside the unit disc, drifting from slice to slice."""
    u = torch.rand((n, 9), generator=gen, dtype=torch.float64).numpy()
    e = np.empty((n, 6))
    e[:, 0:2] = (u[:, 0:2] - 0.5) * 1.1
    e[:, 2:4] = 0.05 + 0.3 * u[:, 2:4]
    e[:, 4] = math.pi * u[:, 4]
    e[:, 5] = -0.3 + 1.3 * u[:, 5]
    return e, (u[:, 6:8] - 0.5) * 0.1


def _lines(g, ell):
    """FP32 line integrals [N_p][N_c] of the ellipses, on the device."""
    hw = 0.5 * max(g.nx, g.ny) * g.pixel_size
    th = torch.as_tensor(g.angles, device="cuda")
    s = (torch.arange(g.n_det, device="cuda", dtype=torch.float64) - g.center).to(torch.float32)
    out = torch.zeros((g.n_angles, g.n_det), device="cuda")
    for x0, y0, a, b, phi, rho in ell:
        x0, y0, a, b = x0 * hw, y0 * hw, a * hw, b * hw
        a2 = (a * torch.cos(th - phi)) ** 2 + (b * torch.sin(th - phi)) ** 2
        s0 = x0 * torch.cos(th) + y0 * torch.sin(th)
        d = s[None, :] - s0.to(torch.float32)[:, None]
        chord = torch.sqrt((a2.to(torch.float32)[:, None] - d * d).clamp_(min=0.0))
        out += chord * (2.0 * rho * a * b / a2).to(torch.float32)[:, None]
    return out


def _sinograms(g, slices, gens):
    cpu, dev = gens
    ell, drift = _ellipses(cpu)
    out = torch.empty((slices, g.n_angles, g.n_det), device="cuda")
    noise = 1e-3 * 0.5 * max(g.nx, g.ny) * g.pixel_size
    for z in range(slices):
        e = ell.copy()
        e[:, 0:2] += drift * (z / max(1, slices - 1))
        torch.randn(out[z].shape, generator=dev, device="cuda", out=out[z])
        out[z] *= noise
        out[z] += _lines(g, e)
    return out


def _images(g, slices, gens):
    """Rasterised ellipses with 5 % noise, FP32 [S][N_y][N_x]."""
    cpu, dev = gens
    ell, drift = _ellipses(cpu)
    hw = 0.5 * max(g.nx, g.ny)
    x = ((torch.arange(g.nx, device="cuda") - 0.5 * (g.nx - 1)) / hw)[None, :]
    y = ((torch.arange(g.ny, device="cuda") - 0.5 * (g.ny - 1)) / hw)[:, None]
    img = torch.randn((slices, g.ny, g.nx), generator=dev, device="cuda") * 0.05
    for z in range(slices):
        for (x0, y0, a, b, phi, rho), (dx, dy) in zip(ell, drift):
            t = z / max(1, slices - 1)
            xr = (x - x0 - t * dx) * math.cos(phi) + (y - y0 - t * dy) * math.sin(phi)
            yr = (y - y0 - t * dy) * math.cos(phi) - (x - x0 - t * dx) * math.sin(phi)
            img[z] += rho * ((xr / a) ** 2 + (yr / b) ** 2 <= 1.0)
    return img


def _counts(g, slices, gens):
    """uint16 projection stack [N_p][S][N_c] with its dark and flat fields."""
    dev = gens[1]
    u = torch.rand((2, slices, g.n_det), generator=dev, device="cuda")
    dark, flat = 90.0 + 20.0 * u[0], 4.5e4 + 1.0e4 * u[1]
    proj = torch.empty((g.n_angles, slices, g.n_det), dtype=torch.int16, device="cuda")
    lines = _sinograms(g, slices, gens)
    kappa = 3.0 / float(lines.max())
    for z in range(slices):
        i = dark[z] + (flat[z] - dark[z]) * torch.exp(-kappa * lines[z])
        proj[:, z] = i.round_().clamp_(0, 65535).to(torch.int32).to(torch.int16)
    return proj.view(torch.uint16), dark, flat


def _ramp(window, n, pitch, length):
    """Real spectrum of the windowed ramp filter on a transform of `length`."""
    d = torch.arange(-(n - 1), n, dtype=torch.float64)

    def ram_lak(m):
        odd = torch.remainder(m, 2) != 0
        h = torch.where(odd, -1.0 / (math.pi * torch.where(odd, m, torch.ones_like(m))) ** 2, torch.zeros_like(m))
        return torch.where(m == 0, torch.full_like(m, 0.25), h)

    if window == "ram_lak":
        h = ram_lak(d)
    elif window == "shepp_logan":
        h = 2.0 / (math.pi ** 2 * (1.0 - 4.0 * d * d))
    else:
        h = 0.5 * ram_lak(d) + 0.25 * (ram_lak(d - 1) + ram_lak(d + 1))
    full = torch.zeros(length, dtype=torch.float64)
    full[torch.remainder(d.to(torch.int64), length)] = h / pitch
    return torch.fft.rfft(full).real.to("cuda")


def _filter(rows, window, dtype):
    """Windowed ramp filter of [S][N_p][N_c] rows in `dtype`, by torch's transforms."""
    n = rows.shape[-1]
    length = 1 << max(6, (2 * n - 2).bit_length())
    spec = _ramp(window, n, 1.0, length).to(dtype)
    out = torch.empty(rows.shape, dtype=dtype, device="cuda")
    per = max(1, (1 << 26) // length)
    flat_in, flat_out = rows.reshape(-1, n), out.reshape(-1, n)
    for i in range(0, flat_in.shape[0], per):
        f = torch.fft.rfft(flat_in[i:i + per].to(dtype), n=length)
        flat_out[i:i + per] = torch.fft.irfft(f * spec, n=length)[:, :n]
    return out


# ---------------------------------------------------------------- passes

def _gens(seed):
    cpu, dev = torch.Generator(), torch.Generator(device="cuda")
    cpu.manual_seed(seed)
    dev.manual_seed(seed)
    return cpu, dev


def prepare(case, seed):
    gens, kind, slabs = _gens(seed), case["kind"], _geometries(case)
    g, s, overlap = slabs[0]
    st = SimpleNamespace(case=case, geom=g, slabs=slabs)
    if kind in ("fbp", "offset", "batch"):
        st.sinos = [_sinograms(gg, ss, gens).to(DTYPES[case["storage"]]) for gg, ss, _ in slabs]
    elif kind == "front":
        st.proj, st.dark, st.flat = _counts(g, s, gens)
    elif kind == "codes":
        st.rows = _filter(_sinograms(g, s, gens), case["window"], torch.float32).to(DTYPES[case["storage"]])
    elif kind == "project":
        st.x = _images(g, s, gens).requires_grad_(True)
        st.seed_grad = _sinograms(g, s, gens)
    else:
        st.x, st.y = _images(g, s, gens), _sinograms(g, s, gens)
    return st


def run(st):
    case, g = st.case, st.geom
    kind = case["kind"]
    if kind == "fbp":
        return xct.fbp(st.sinos[0], g, case["window"], DTYPES[case["filtered"]])
    if kind == "offset":
        return xct.fbp_offset(st.sinos[0], g, case["window"], case["overlap"], DTYPES[case["filtered"]])
    if kind == "batch":
        images = [torch.empty((s, gg.ny, gg.nx), device="cuda") for gg, s, _ in st.slabs]
        xct.xct_fbp_batch([(gg, q, f) for (gg, _, _), q, f in zip(st.slabs, st.sinos, images)],
                          case["window"], DTYPES[case["filtered"]])
        return images
    if kind == "front":
        out = torch.empty((case["slices"], g.n_angles, g.n_det), device="cuda")
        xct.xct_preprocess_filter(g, st.proj, st.dark, st.flat, 0, out, case["window"], FLOOR, case["sigma"])
        return out
    if kind == "codes":
        out = torch.empty((case["slices"], g.ny, g.nx), dtype=torch.uint16, device="cuda")
        xct.xct_backproject_u16(g, st.rows, out, math.pi / g.n_angles, CODE_WATER, CODE_MIN, CODE_MAX)
        return out.view(torch.int16)  # the same 16 bits, in a type that torch indexes on the device
    if kind == "project":
        y = xct.project(st.x, g)
        (gx,) = torch.autograd.grad(y, st.x, st.seed_grad)
        return {"y": y.detach(), "grad": gx}
    r, grad = torch.empty_like(st.y), torch.empty_like(st.x)
    xct.xct_forward_residual(g, st.x, st.y, r)
    xct.xct_project_adjoint(g, r, grad)
    return {"r": r, "grad": grad}


def work(case):
    """Inputs read once, outputs written once; 6 operations per voxel update
    (coordinate, interpolation, accumulation), 5 n log2 n per transform."""
    kind, s = case["kind"], case["slices"]
    b, f = 0.0, 0.0
    for g, sl, overlap in _geometries(case):
        rows, image, updates = float(sl) * g.n_angles * g.n_det, float(sl) * g.nx * g.ny, float(sl) * g.nx * g.ny * g.n_angles
        length = 1 << (2 * g.n_det - 2).bit_length()
        transform = 2.0 * 2.5 * length * math.log2(length) * sl * g.n_angles
        if kind in ("fbp", "offset", "batch"):
            b += rows * SIZE[case["storage"]] + 4.0 * image
            f += 6.0 * updates + transform
        elif kind == "front":
            b += rows * (2 + 4) + 8.0 * s * g.n_det
            f += transform + rows * (10 + 2 * (2 * int(4 * case["sigma"] + 0.5) + 1))
        elif kind == "codes":
            b += rows * SIZE[case["storage"]] + 2.0 * image
            f += 6.0 * updates
        else:
            b += 4.0 * (2 * rows + 2 * image)
            f += 12.0 * updates
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------- 64-bit values

def _coords(g):
    x = (torch.arange(g.nx, device="cuda", dtype=torch.float64) - 0.5 * (g.nx - 1)) * g.pixel_size
    y = (torch.arange(g.ny, device="cuda", dtype=torch.float64) - 0.5 * (g.ny - 1)) * g.pixel_size
    return x[None, :], y[:, None]


def _taps(g, th, x, y):
    u = x * math.cos(th) + y * math.sin(th) + g.center
    n = torch.floor(u)
    # left tap in a row with two zero bins on either side of the detector
    return (n.to(torch.int64) + 2).clamp_(0, g.n_det + 2).reshape(-1), (u - n).reshape(-1)


def _transpose(g, rows, scale):
    """scale * A^T rows, FP64."""
    x, y = _coords(g)
    s = rows.shape[0]
    img = torch.zeros((s, g.ny * g.nx), dtype=torch.float64, device="cuda")
    for k, th in enumerate(g.angles.tolist()):
        i, t = _taps(g, th, x, y)
        row = torch.zeros((s, g.n_det + 4), dtype=torch.float64, device="cuda")
        row[:, 2:g.n_det + 2] = rows[:, k]
        step = row[:, 1:] - row[:, :-1]
        for z in range(s):
            img[z] += row[z][i] + t * step[z][i]
    return (img * scale).reshape(s, g.ny, g.nx)


def _forward(g, img):
    """(pixel^2 / pitch) A img, FP64."""
    x, y = _coords(g)
    s = img.shape[0]
    out = torch.zeros((s, g.n_angles, g.n_det), dtype=torch.float64, device="cuda")
    flat = img.to(torch.float64).reshape(s, -1)
    edges = torch.arange(g.n_det + 4, device="cuda")
    for k, th in enumerate(g.angles.tolist()):
        # sums over the pixels of each bin, from running sums over the pixels in bin order
        i, t = _taps(g, th, x, y)
        i, order = torch.sort(i)
        v = flat[:, order]
        right = v * t[order]
        at = torch.searchsorted(i, edges)
        parts = []
        for w in (v - right, right):
            run_sum = torch.cumsum(w, dim=1)
            total = torch.cat([torch.zeros((s, 1), dtype=torch.float64, device="cuda"), run_sum], dim=1)[:, at]
            parts.append(total[:, 1:] - total[:, :-1])  # by left tap
        out[:, k] = parts[0][:, 2:g.n_det + 2] + parts[1][:, 1:g.n_det + 1]
    return out * g.pixel_size ** 2


def _front_rows(case, g, proj, dark, flat):
    i = proj.view(torch.int16).to(torch.int32).bitwise_and_(0xFFFF).to(torch.float64).permute(1, 0, 2)
    d, f = dark.to(torch.float64)[:, None], flat.to(torch.float64)[:, None]
    p = -torch.log((i - d).clamp(min=FLOOR) / (f - d).clamp(min=FLOOR))
    sigma = case["sigma"]
    if sigma > 0:
        r = int(4 * sigma + 0.5)
        w = [math.exp(-0.5 * (m / sigma) ** 2) for m in range(-r, r + 1)]
        at = torch.arange(g.n_det, device="cuda")
        p = sum(v / sum(w) * p[:, :, (at + m).clamp(0, g.n_det - 1)] for m, v in zip(range(-r, r + 1), w))
    return p


def _offset_rows(case, g, sino):
    """Redundancy-weighted rows on the mirrored detector, and its geometry."""
    c, nc = g.center, g.n_det
    right = (nc - 1) - c >= c
    n_virtual = int(2 * (nc - 1 - c) + 1 if right else 2 * c + 1)
    center = float(nc - 1 - c if right else c)
    first = int(n_virtual - nc if right else 0)
    t = (torch.arange(nc, device="cuda", dtype=torch.float64) - c) * (1.0 if right else -1.0) / case["overlap"]
    w = torch.sin(0.25 * math.pi * (1.0 + t.clamp(-1.0, 1.0))) ** 2
    rows = torch.zeros((sino.shape[0], g.n_angles, n_virtual), dtype=torch.float64, device="cuda")
    rows[:, :, first:first + nc] = sino.to(torch.float64) * w
    return rows, SimpleNamespace(**{**vars(g), "n_det": n_virtual, "center": center})


def exact(case, seed):
    kind = case["kind"]
    if kind == "codes" or (kind != "front" and _updates(case) > EXACT_UPDATES):
        return None
    st = prepare(case, seed)
    g = st.geom
    if kind == "front":
        rows = _front_rows(case, g, st.proj, st.dark, st.flat)
        return _filter(rows, case["window"], torch.float64)
    if kind in ("fbp", "batch"):
        imgs = [_transpose(gg, _filter(q, case["window"], torch.float64), math.pi / gg.n_angles)
                for (gg, _, _), q in zip(st.slabs, st.sinos)]
        return imgs if kind == "batch" else imgs[0]
    if kind == "offset":
        rows, gv = _offset_rows(case, g, st.sinos[0])
        return _transpose(gv, _filter(rows, case["window"], torch.float64), 2.0 * math.pi / g.n_angles)
    if kind == "project":
        return {"y": _forward(g, st.x.detach()), "grad": _transpose(g, st.seed_grad.to(torch.float64), g.pixel_size ** 2)}
    r = st.y.to(torch.float64) - _forward(g, st.x)
    return {"r": r, "grad": _transpose(g, r, g.pixel_size ** 2)}
