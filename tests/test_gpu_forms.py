"""GPU tests of where one call takes one kernel form or another: which slabs
the matrix cores hold, and what a form must not change for the caller."""

import math

import numpy as np
import pytest
import torch

import oracle
import synth
from tests.gpu_util import rel_l2, say, to_dev

pytestmark = pytest.mark.gpu

# The gate of the vector kernels: coordinates below 96 or 192 bins; and of the
# matrix cores, below 64 (FP32 sums into an image of the same size besides).
TOL = 2e-5
TOL_MATRIX = 1e-5


@pytest.fixture(scope="module")
def xct():
    import paper_2505_13955_amd as pkg

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    pkg.load_library()
    return pkg


def on_matrix_cores(xct, g, S, filtered=torch.float32, rows=None):
    """Partial images of a call of this slab alone on the matrix cores (0 or 2 to
    64), None if it is not there: the workspace behind the counters, the
    descriptor and the rows holds the magnitudes, the split table (of `rows`
    angles where it does not hold all) and that many images."""
    a256 = lambda b: (b + 255) // 256 * 256
    size = 4 if filtered == torch.float32 else 2
    sino = torch.empty((S, g.n_angles, g.n_det), device="cuda")
    scratch = xct.xct_fbp_workspace_bytes([(g, sino, None)], filtered) - 512 - a256(sino.numel() * size)
    rest = scratch - a256(4 * (2 * S + 1)) - a256((S + 3) // 4 * (rows or g.n_angles) * g.n_det * 16)
    fit = [p for p in [0] + list(range(2, 65)) if rest == a256(p * 4 * S * g.nx * g.ny)]
    return fit[0] if fit else None


def sampled(q, g, pixels, scale):
    """FP64 back-projection of the rows q (S, N_p, N_c) at pixels (n, 2) of every slice."""
    x = (pixels[:, 1].double() - 0.5 * (g.nx - 1)) * g.pixel_size
    y = (pixels[:, 0].double() - 0.5 * (g.ny - 1)) * g.pixel_size
    out = torch.zeros((q.shape[0], len(pixels)), dtype=torch.float64, device=q.device)
    th = torch.as_tensor(np.asarray(g.angles), device=q.device)
    for k in range(0, g.n_angles, 1024):
        t = th[k:k + 1024, None]
        u = (x * torch.cos(t) + y * torch.sin(t)) / g.det_pitch + g.center
        n = torch.floor(u)
        f, n = u - n, n.long()
        for z in range(q.shape[0]):
            for bin_, w in ((n, 1.0 - f), (n + 1, f)):
                inside = (bin_ >= 0) & (bin_ < g.n_det)
                v = torch.gather(q[z, k:k + 1024].double(), 1, bin_.clamp(0, g.n_det - 1))
                out[z] += torch.where(inside, v * w, 0.0).sum(0)
    return out * scale


def random_pixels(g, n, seed):
    gen = torch.Generator().manual_seed(seed)
    return torch.stack([torch.randint(g.ny, (n,), generator=gen), torch.randint(g.nx, (n,), generator=gen)], 1).cuda()


@pytest.mark.parametrize("case", [
    # slices, nx, ny, angles, bins, centre
    (61, 413, 390, 301, 600, 299.7),    # plain
    (4, 813, 811, 602, 1160, 579.5),    # mirror with reflection
    (8, 1030, 1030, 300, 1460, 729.5),  # quarter turn
])
def test_wide_range_of_magnitudes(xct, case):
    """Samples far smaller than the slice's largest keep their bits: a disc of
    pixels that sees nothing but columns 2^-e as large as the rest, and every
    pixel that one huge bin's ray does not meet."""
    S, nx, ny, na, nd, c = case
    g = synth.Geometry(n_angles=na, n_det=nd, nx=nx, ny=ny, center=c)
    assert on_matrix_cores(xct, g, S) is not None
    rng = np.random.default_rng(61)
    q = rng.standard_normal((S, na, nd)).astype(np.float32)
    inner = np.abs(np.arange(nd) - c) <= 70
    x, y = np.arange(nx) - 0.5 * (nx - 1), np.arange(ny) - 0.5 * (ny - 1)
    disc = x[None, :] ** 2 + y[:, None] ** 2 <= 67.0 ** 2
    parts = [np.where(inner, q, 0.0), np.where(inner, 0.0, q)]
    ref_in, ref_out = (oracle.backproject(p.astype(np.float64), g, oracle.adjoint_scale(g)) for p in parts)
    assert np.all(ref_out[:, disc] == 0.0)
    for e in (0, 17, 22, 40):  # 17: still within what the split holds
        say("wide range", case, e)
        img = xct.project_adjoint(to_dev(parts[0] * np.float32(2.0 ** -e) + parts[1]), g).cpu().numpy()
        ref = ref_in * 2.0 ** -e + ref_out
        for z in range(S):
            assert rel_l2(img[z][disc], ref[z][disc]) < TOL, (e, z)
            assert rel_l2(img[z], ref[z]) < TOL, (e, z)
    k, n, z = na // 3, int(c) + 40, S - 1
    hot = q.copy()
    hot[z, k, n] = 1e10
    say("one huge bin", case)
    img = xct.project_adjoint(to_dev(hot), g).cpu().numpy()
    off = np.abs(x[None, :] * math.cos(g.angles[k]) + y[:, None] * math.sin(g.angles[k]) + c - n) > 1.001
    ref = ref_in + ref_out
    for s in range(S):
        at = off if s == z else np.ones_like(off)
        assert rel_l2(img[s][at], ref[s][at]) < TOL, s


def captured(fn):
    """fn() captured into a graph, on the side stream that the capture uses."""
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fn()
    return graph


@pytest.mark.parametrize("case", [
    # slices, side, angles, bins, centre: what an eager call projects from
    (1, 512, 720, 730, 364.5),    # turned copies
    (2, 512, 96, 730, 361.7),     # the same, two slices
    (1, 200, 90, 290, 144.5),     # the slice itself, walks in parts
])
def test_forward_projection_captured_after_an_eager_call(xct, case):
    """A geometry that has been projected once can be captured, whichever form
    the eager call took: replays equal the eager sinogram within rounding, and
    each other to the bit."""
    S, n, na, nd, c = case
    g = synth.Geometry(n_angles=na, n_det=nd, nx=n, ny=n, center=c)
    x = torch.randn((S, n, n), generator=torch.Generator().manual_seed(n)).cuda()
    y = torch.randn((S, na, nd), generator=torch.Generator().manual_seed(na)).cuda()
    say("captured forward", case)
    want = xct.forward_project(x, g)
    p, r = torch.empty_like(want), torch.empty_like(want)

    def pair():
        xct.xct_forward_project(g, x, p)
        xct.xct_forward_residual(g, x, y, r)

    graph = captured(pair)
    for k in range(3):
        x.copy_(torch.randn(x.shape, generator=torch.Generator().manual_seed(k)))
        want = xct.forward_project(x, g)
        graph.replay()
        torch.cuda.synchronize()
        assert rel_l2(p.cpu().numpy(), want.cpu().double().numpy()) < TOL
        assert rel_l2(r.cpu().numpy(), (y.double() - want.double()).cpu().numpy()) < TOL
        first = p.clone()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(p, first)


@pytest.mark.parametrize("case", [
    # slabs, slices, nx, ny, angles, bins: what a slab alone takes
    (140, 1, 256, 256, 90, 367),    # parts
    (14, 14, 400, 300, 500, 520),   # the matrix cores
])
def test_batch_that_fills_the_device_walks_whole(xct, case):
    """Slabs that alone are split, or on the matrix cores, because they would
    leave the device idle: in a batch that fills it they are walked whole by the
    vector kernels, as xct_backproject walks them, to the bit."""
    n, S, nx, ny, na, nd = case
    g = synth.Geometry(n_angles=na, n_det=nd, nx=nx, ny=ny, center=(nd - 1) / 2.0)
    assert (on_matrix_cores(xct, g, S) is None) == (S == 1)
    p = torch.randn((n, S, na, nd), generator=torch.Generator().manual_seed(na)).cuda()
    img = torch.empty((n, S, ny, nx), device="cuda")
    say("full batch", case)
    xct.xct_fbp_batch([(g, p[i], img[i]) for i in range(n)], "hann")
    q = torch.empty_like(p[0])
    want = torch.empty_like(img[0])
    for i in (0, 1, n // 2, n - 1):
        xct.xct_filter(g, p[i], q, "hann")
        xct.xct_backproject(g, q, want, math.pi / na)
        torch.cuda.synchronize()
        assert torch.equal(want, img[i]), i
        alone = xct.fbp(p[i], g, "hann")
        assert rel_l2(alone.cpu().numpy(), img[i].cpu().double().numpy()) < TOL
    ref = oracle.fbp(p[n - 1].double().cpu().numpy(), g, "hann")
    assert rel_l2(img[n - 1].cpu().numpy(), ref) < TOL


@pytest.mark.parametrize("case", [
    # slices, side, angles, bins: what an eager call takes
    (1, 256, 360, 367),    # parts
    (4, 512, 720, 727),    # parts
    (4, 813, 602, 1160),   # the matrix cores
])
def test_adjoint_captured_after_an_eager_call(xct, case):
    """Under capture there is no scratch: whole walks of the vector kernels, as
    xct_backproject takes them below its limit, to the bit."""
    S, n, na, nd = case
    g = synth.Geometry(n_angles=na, n_det=nd, nx=n, ny=n, center=(nd - 1) / 2.0)
    q = torch.randn((S, na, nd), generator=torch.Generator().manual_seed(n)).cuda()
    say("captured adjoint", case)
    img = xct.project_adjoint(q, g)
    graph = captured(lambda: xct.xct_project_adjoint(g, q, img))
    want = torch.empty_like(img)
    for k in range(3):
        q.copy_(torch.randn(q.shape, generator=torch.Generator().manual_seed(k)))
        eager = xct.project_adjoint(q, g)
        graph.replay()
        xct.xct_backproject(g, q, want, 1.0)
        torch.cuda.synchronize()
        assert torch.equal(img, want)
        assert rel_l2(img.cpu().numpy(), eager.cpu().double().numpy()) < TOL


@pytest.mark.parametrize("case", [
    # slices, nx, ny, angles, bins, centre: more items than workgroups, no multiple of the XCDs
    (72, 576, 576, 240, 815, 407.0),    # symmetric
    (37, 500, 460, 401, 681, 340.0),    # mirror
    (3, 1301, 1203, 301, 1800, 899.0),  # mirror, few slices
])
def test_non_finite_slab_of_many_items(xct, case):
    """A slab that leaves the matrix cores for a non-finite element is walked
    as xct_backproject walks it below its limit, to the bit."""
    S, nx, ny, na, nd, c = case
    g = synth.Geometry(n_angles=na, n_det=nd, nx=nx, ny=ny, center=c)
    assert on_matrix_cores(xct, g, S) is not None
    q = torch.randn((S, na, nd), generator=torch.Generator().manual_seed(nx)).cuda()
    q[0, na // 2, nd // 3] = float("inf")
    say("non-finite, many items", case)
    img = xct.project_adjoint(q, g)
    want = torch.empty_like(img)
    xct.xct_backproject(g, q, want, 1.0)
    torch.cuda.synchronize()
    assert not torch.isfinite(img[0]).all() and torch.isfinite(img[1:]).all()
    assert torch.equal(img.nan_to_num(0.5, 7.0, -7.0), want.nan_to_num(0.5, 7.0, -7.0))


PLAIN, MIRROR, MIRROR2, QUARTER, QUARTER2 = range(5)


@pytest.mark.parametrize("case", [
    # columns, kind, partial images; slices, nx, ny, angles, bins, centre, angle set
    (16, PLAIN, 0, 8, 713, 690, 180, 1034, 516.3, "half"),
    (16, PLAIN, 2, 15, 433, 410, 301, 636, 317.3, "half"),
    (32, PLAIN, 0, 31, 713, 690, 101, 1034, 516.3, "half"),
    (32, PLAIN, 5, 31, 313, 290, 600, 466, 232.3, "half"),
    (64, PLAIN, 2, 61, 313, 290, 404, 466, 232.3, "half"),
    (16, MIRROR, 0, 7, 602, 591, 180, 857, 428.0, "half"),
    (16, MIRROR, 5, 8, 300, 289, 600, 429, 214.0, "half"),
    (32, MIRROR, 0, 31, 700, 689, 101, 997, 498.0, "half"),
    (32, MIRROR, 3, 16, 513, 502, 1001, 731, 365.0, "rand"),
    (64, MIRROR, 2, 61, 300, 289, 404, 429, 214.0, "half"),
    (16, MIRROR2, 0, 3, 1020, 1009, 180, 1451, 725.0, "half"),
    (32, MIRROR2, 3, 7, 813, 802, 301, 1157, 578.0, "half"),
    (64, MIRROR2, 3, 15, 513, 502, 600, 731, 365.0, "half"),
    (16, QUARTER, 0, 31, 300, 300, 180, 429, 214.0, "full"),
    (32, QUARTER, 5, 15, 420, 420, 600, 599, 299.0, "half"),
    (64, QUARTER, 2, 15, 602, 602, 404, 857, 428.0, "half"),
    (64, QUARTER, 0, 61, 420, 420, 404, 599, 299.0, "full"),
    (32, QUARTER2, 0, 3, 1950, 1950, 180, 2772, 1385.5, "half"),
    (64, QUARTER2, 0, 7, 1400, 1400, 404, 1991, 995.0, "half"),
])
def test_matrix_kernels(xct, case):
    """Every kind and column count of the matrix-core kernel, with the kernel
    that ran read from a trace."""
    cols, kind, images, S, nx, ny, na, nd, c, angles = case
    rng = np.random.default_rng(cols + kind)
    th = rng.uniform(-math.pi, 2.0 * math.pi, na) if angles == "rand" else np.arange(na) * ((2.0 if angles == "full" else 1.0) * math.pi / na)
    g = synth.Geometry(n_angles=na, n_det=nd, nx=nx, ny=ny, center=c, angles=th)
    q = torch.randn((S, na, nd), generator=torch.Generator().manual_seed(na)).cuda()
    base = torch.randn((S, ny, nx), generator=torch.Generator().manual_seed(nd)).cuda()
    say("matrix kernel", case)
    img = xct.project_adjoint(q, g)
    acc = base.clone()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as trace:
        xct.xct_project_adjoint(g, q, acc, -0.5, accumulate=True)
        torch.cuda.synchronize()
    ran = [e.name for e in trace.events() if "bp_mfma" in e.name]
    assert ran and all(f"<{cols}, {kind}>" in name for name in ran), ran
    at = random_pixels(g, 3000, nx)
    ref = sampled(q, g, at, 1.0)
    for z in range(S):
        assert rel_l2(img[z, at[:, 0], at[:, 1]].cpu(), ref[z].cpu()) < TOL_MATRIX, z
        assert rel_l2((acc - base)[z, at[:, 0], at[:, 1]].cpu(), -0.5 * ref[z].cpu()) < TOL_MATRIX, z
    if angles != "full":  # (a launch of a full turn's set makes the table of that set)
        assert on_matrix_cores(xct, g, S) == images


@pytest.mark.parametrize("filtered", [torch.float32, torch.float16, torch.bfloat16])
def test_batch_of_matrix_and_split_slabs(xct, filtered):
    """A slab on the matrix cores, one with partial images there, and slabs
    whose angles are split, in one batch: their scratch takes turns, and every
    image equals its own call's to the bit; also the rows in 16 bits."""
    slabs = []
    for i, (S, nx, ny, na, nd, c, images) in enumerate([
            (1, 256, 256, 360, 367, 183.0, None),      # split
            (4, 813, 811, 602, 1160, 579.5, 3),        # mirror with reflection
            (3, 131, 77, 163, 150, 74.3, None),        # split, a pair and one
            (64, 512, 500, 150, 729, 363.7, 0),        # plain
            (8, 1030, 1030, 300, 1460, 729.5, 2)]):    # quarter turn
        g = synth.Geometry(n_angles=na, n_det=nd, nx=nx, ny=ny, center=c)
        assert on_matrix_cores(xct, g, S, filtered) == images, i
        p = torch.randn((S, na, nd), generator=torch.Generator().manual_seed(i)).cuda()
        slabs.append((g, p, torch.full((S, ny, nx), float("nan"), device="cuda")))
    say("batch of matrix and split slabs", filtered)
    xct.xct_fbp_batch(slabs, "hann", filtered)
    for i, (g, p, img) in enumerate(slabs):
        alone = xct.fbp(p, g, "hann", filtered)
        rows = xct.filter(p, g, "hann", filtered)
        torch.cuda.synchronize()
        assert torch.equal(alone, img), i
        at = random_pixels(g, 3000, i)
        assert rel_l2(img[:, at[:, 0], at[:, 1]].cpu(), sampled(rows, g, at, math.pi / g.n_angles).cpu()) < TOL, i


@pytest.mark.parametrize("case", [
    # slabs, and the launches that sum their copies: 64 images a launch
    ([(1, 40, 41, 400)] * 70, 2),
    # the copies that these ask for alone are more than there is room for
    ([(1, 1200, 1200, 900 + 40 * i) for i in range(5)] + [(1, 64, 64, 3000), (3, 300, 250, 200)], 1)])
def test_batch_of_split_slabs(xct, case):
    """Slabs of fractional axis that a batch splits: their copies are summed
    together, the room for copies goes to the longest walks and the other
    slabs walk whole; against separate calls (sums in another order: some
    sqrt(angles) roundings of 2^-24)."""
    sizes, launches = case
    slabs, asked = [], 0
    for i, (S, nx, ny, na) in enumerate(sizes):
        nd = int(1.42 * max(nx, ny)) + 6
        g = synth.Geometry(n_angles=na, n_det=nd, nx=nx, ny=ny, center=(nd - 1) / 2 + 0.3)
        p = torch.randn((S, na, nd), generator=torch.Generator().manual_seed(i)).cuda()
        slabs.append((g, p, torch.full((S, ny, nx), float("nan"), device="cuda")))
        asked += xct.xct_fbp_workspace_bytes(slabs[-1:])
    if len(sizes) < 64:
        assert xct.xct_fbp_workspace_bytes(slabs) < asked - (64 << 20)
    say("batch of split slabs", len(sizes))
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as trace:
        xct.xct_fbp_batch(slabs, "hann")
        torch.cuda.synchronize()
    assert len([e for e in trace.events() if "sum_" in e.name and "kernel" in e.name]) == launches
    alone = [xct.fbp(p, g, "hann") for g, p, img in slabs]
    for i, (g, p, img) in enumerate(slabs):
        assert rel_l2(img.cpu(), alone[i].cpu()) < 5e-6, i
    # without room for the copies every slab walks whole
    ws = torch.empty(xct.xct_fbp_workspace_bytes(slabs) - 256, dtype=torch.uint8, device="cuda")
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as trace:
        xct.xct_fbp_batch(slabs, "hann", workspace=ws)
        torch.cuda.synchronize()
    assert not [e for e in trace.events() if "sum_" in e.name and "kernel" in e.name]
    for i, (g, p, img) in enumerate(slabs):
        assert rel_l2(img.cpu(), alone[i].cpu()) < 5e-6, i


@pytest.mark.parametrize("storage", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("nx, ny, na, nd", [
    (1024, 1024, 1024, 1449),  # quarter turn
    (1025, 1001, 1023, 1449),  # mirror; rows of a slice not 16-byte aligned
])
def test_back_projection_of_stored_rows(xct, storage, nx, ny, na, nd):
    """xct_backproject from 1.5e10 updates, rows in every storage type; with a
    non-finite element pixels off its ray are as before within rounding."""
    S = 16
    g = synth.Geometry(n_angles=na, n_det=nd, nx=nx, ny=ny, center=(nd - 1) / 2.0)
    size = torch.float32 if storage == torch.float32 else torch.float16
    assert on_matrix_cores(xct, g, S, size) is not None and S * na * nx * ny >= 1.5e10
    q = torch.randn((S, na, nd), generator=torch.Generator().manual_seed(nd)).cuda().to(storage)
    say("stored rows", storage, na)
    img = xct.backproject(q, g, 0.25)
    at = random_pixels(g, 3000, 3)
    ref = sampled(q, g, at, 0.25)
    got = img[:, at[:, 0], at[:, 1]].double()
    for z in range(S):
        assert rel_l2(got[z].cpu(), ref[z].cpu()) < TOL, z
    for bad in (float("nan"), float("inf")):
        q[3, na // 3, nd // 2] = bad
        hit = xct.backproject(q, g, 0.25)[:, at[:, 0], at[:, 1]].double()
        torch.cuda.synchronize()
        finite = torch.isfinite(hit)
        x, y = at[:, 1] - 0.5 * (nx - 1), at[:, 0] - 0.5 * (ny - 1)
        off = (x * math.cos(g.angles[na // 3]) + y * math.sin(g.angles[na // 3]) + g.center - nd // 2).abs()
        assert not finite[3][off < 0.99].any() and finite[3][off > 1.01].all()
        assert finite[[z for z in range(S) if z != 3]].all()
        assert rel_l2(hit[finite].cpu(), ref[finite].cpu()) < TOL


@pytest.mark.parametrize("case", [
    # slices, nx, ny, angles, bins, centre, rows of a split table, partial images
    (32, 1024, 1024, 2049, 4100, 2049.3, 1028, 0),   # plain
    (32, 1024, 1024, 2049, 4100, 2049.5, 1028, 0),   # mirror
    (3, 1500, 1499, 8201, 8190, 4094.5, 4104, 4),    # mirror, each range's parts items of their own
    (3, 900, 900, 8200, 8190, 4094.5, 4104, 2),      # the same, quarter turn
])
def test_split_table_in_ranges(xct, case):
    """Split tables beyond 1 GiB are made and used range by range of angles, the
    image accumulating; the last range is shorter."""
    S, nx, ny, na, nd, c, rows, images = case
    g = synth.Geometry(n_angles=na, n_det=nd, nx=nx, ny=ny, center=c)
    assert on_matrix_cores(xct, g, S, rows=rows) == images
    q = torch.randn((S, na, nd), device="cuda", generator=torch.Generator(device="cuda").manual_seed(na))
    base = torch.randn((S, ny, nx), device="cuda", generator=torch.Generator(device="cuda").manual_seed(nd))
    say("ranges", case)
    img = xct.project_adjoint(q, g)
    acc = base.clone()
    xct.xct_project_adjoint(g, q, acc, -0.5, accumulate=True)
    at = random_pixels(g, 1500, nx)
    ref = sampled(q, g, at, 1.0)
    got = img[:, at[:, 0], at[:, 1]].double()
    added = (acc - base)[:, at[:, 0], at[:, 1]].double()
    for z in range(S):
        assert rel_l2(got[z].cpu(), ref[z].cpu()) < TOL, z
        assert rel_l2(added[z].cpu(), -0.5 * ref[z].cpu()) < TOL, z


@pytest.mark.parametrize("S, nx, ny, na, nd, c", [
    (9, 700, 700, 800, 991, 495.0),      # symmetric
    (9, 801, 702, 701, 1135, 567.0),     # mirror, more items than two rounds
    (5, 1100, 1000, 601, 1557, 777.7),   # generic
    (8, 1408, 1408, 1024, 1992, 995.5),  # from 1.5e10 updates: the image on the matrix cores
])
def test_codes_against_the_image(xct, S, nx, ny, na, nd, c):
    """Codes are the documented rounding of xct_backproject's image below 1.5e10
    updates, and within one code of it where that image takes other kernels."""
    g = synth.Geometry(n_angles=na, n_det=nd, nx=nx, ny=ny, center=c)
    water, lo, hi = 0.3, -1000.0, 4000.0
    q = torch.randn((S, na, nd), generator=torch.Generator().manual_seed(nx)).cuda()
    scale = 0.3 / math.sqrt(na)
    codes = torch.empty((S, ny, nx), dtype=torch.uint16, device="cuda")
    image = torch.empty((S, ny, nx), device="cuda")
    say("codes", nx, na)
    xct.xct_backproject_u16(g, q, codes, scale, water, lo, hi)
    xct.xct_backproject(g, q, image, scale)
    torch.cuda.synchronize()
    span = 65535.0 / (hi - lo)
    a, b = np.float32(1000.0 / water * span), np.float32((-1000.0 - lo) * span)
    mu = image.cpu().numpy()
    want = np.clip(np.rint(mu * a + b), 0, 65535).astype(np.int64)
    off = np.abs(codes.cpu().numpy().astype(np.int64) - want)
    assert (want > 0).mean() > 0.3 and (want < 65535).mean() > 0.3
    if S * na * nx * ny < 1.5e10:
        assert off.max() == 0
    else:
        assert on_matrix_cores(xct, g, S) is not None
        # (images 5e-6 apart, 11,000 codes of spread: some 0.04 codes on average)
        assert off.max() <= 1 and (off > 0).mean() < 0.1


def test_batch_captured_after_an_eager_call(xct):
    """A batch takes the same forms under capture: its scratch is the caller's."""
    slabs = []
    for i, (S, nx, ny, na, nd, c) in enumerate([(1, 256, 256, 360, 367, 183.0), (4, 813, 811, 602, 1160, 579.5),
                                                (2, 131, 77, 163, 150, 74.3)]):
        g = synth.Geometry(n_angles=na, n_det=nd, nx=nx, ny=ny, center=c)
        p = torch.randn((S, na, nd), generator=torch.Generator().manual_seed(i)).cuda()
        slabs.append((g, p, torch.empty((S, ny, nx), device="cuda")))
    ws = torch.empty(xct.xct_fbp_workspace_bytes(slabs), dtype=torch.uint8, device="cuda")
    say("captured batch")
    xct.xct_fbp_batch(slabs, "hann", workspace=ws)
    graph = captured(lambda: xct.xct_fbp_batch(slabs, "hann", workspace=ws))
    for k in range(3):
        for i, (_, p, _) in enumerate(slabs):
            p.copy_(torch.randn(p.shape, generator=torch.Generator().manual_seed(10 * k + i)))
        want = [torch.empty_like(img) for _, _, img in slabs]
        xct.xct_fbp_batch([(g, p, w) for (g, p, _), w in zip(slabs, want)], "hann")
        graph.replay()
        torch.cuda.synchronize()
        for (_, _, img), w in zip(slabs, want):
            assert torch.equal(img, w)
