"""GPU parity of the back-projector's matrix-core form and of calls whose
angles are split into parts, against the FP64 oracle.

The adjoint and the batch choose the form from the call's size alone; the
sizes here lie where each kind is chosen: plain, mirror and quarter-turn
columns, each with and without the reflection, one and two 32-column tiles,
slice counts that are no multiple of a group of four, ragged tiles and angle
counts, arbitrary angles, and small calls split over the device."""

import math

import numpy as np
import pytest
import torch

import oracle
import synth
from tests.gpu_util import rel_l2, say, to_dev

pytestmark = pytest.mark.gpu

# Coordinates are FP32 below 64 bins (2^-19 bin of rounding, some three of them
# per pixel and angle); white-noise rows have a slope of sqrt(2) of their
# magnitude per bin, and interpolation keeps sqrt(2/3) of it: 3 2^-19 sqrt(3) =
# 1.0e-5.
TOL = 1e-5
# The vector kernels' gate (coordinates below 96 or 192 bins)
TOL_VECTOR = 2e-5


@pytest.fixture(scope="module")
def xct():
    import paper_2505_13955_amd as pkg

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    pkg.load_library()
    return pkg


def _angles(kind, n, rng):
    if kind == "rand":
        return rng.uniform(-math.pi, 2 * math.pi, n)
    return np.arange(n) * ((2.0 if kind == "full" else 1.0) * math.pi / n)


CASES = [
    # slices, nx, ny, angles, bins, centre, pixel, angle set
    (70, 64, 64, 133, 70, 31.7, 1.0, "half"),      # plain
    (37, 120, 90, 151, 150, 74.3, 1.1, "rand"),    # plain, arbitrary angles, largest pixel
    (33, 101, 99, 249, 150, 74.5, 1.0, "half"),    # mirror, odd sizes
    (35, 130, 64, 120, 160, 80.0, 0.8, "rand"),    # mirror, arbitrary angles
    (5, 200, 200, 101, 289, 144.0, 1.0, "half"),   # mirror with reflection
    (7, 321, 257, 361, 461, 230.0, 1.0, "half"),   # the same, middle row and column
    (8, 512, 512, 360, 727, 363.0, 1.0, "half"),   # quarter turn with reflection
    (12, 300, 300, 180, 427, 213.0, 1.0, "half"),  # quarter turn, ragged quadrant
    (18, 258, 258, 128, 300, 149.5, 1.0, "full"),  # quarter turn, two half-turn sets
    (1, 256, 256, 360, 367, 183.0, 1.0, "half"),   # split, vector kernels: symmetric
    (3, 131, 77, 163, 150, 80.0, 1.1, "half"),     # split: mirror
    (1, 200, 70, 200, 290, 144.6, 1.4, "rand"),    # split: generic
    (2, 256, 256, 512, 367, 183.0, 1.0, "full"),   # split: symmetric, parts across the two sets
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_adjoint_matches_oracle(xct, case):
    S, nx, ny, na, nd, c, px, kind = CASES[case]
    rng = np.random.default_rng(900 + case)
    g = synth.Geometry(n_angles=na, n_det=nd, nx=nx, ny=ny, center=c, pixel_size=px, angles=_angles(kind, na, rng))
    q = rng.standard_normal((S, na, nd)) * np.linspace(0.5, 2.0, S)[:, None, None]
    base = rng.standard_normal((S, ny, nx))
    say("adjoint", CASES[case])
    dq = to_dev(q)
    img = xct.project_adjoint(dq, g)
    acc = to_dev(base)
    xct.xct_project_adjoint(g, dq, acc, -0.5, accumulate=True)
    torch.cuda.synchronize()
    ref = oracle.backproject(q.astype(np.float32).astype(np.float64), g, oracle.adjoint_scale(g))
    for z in range(S):
        assert rel_l2(img[z].cpu().numpy(), ref[z]) < TOL, z
    assert rel_l2(acc.cpu().numpy() - base.astype(np.float32), -0.5 * ref) < TOL


@pytest.mark.parametrize("case", [
    # slices, nx, ny, angles, bins, centre, pixel, angle set
    # ragged tiles and slice groups, most with parts of their own
    (16, 700, 300, 501, 770, 383.1, 0.07, "half"),   # plain, the image within a few bins
    (30, 515, 490, 301, 729, 363.7, 1.1, "rand"),    # the largest pixel
    (61, 413, 390, 301, 600, 299.7, 1.0, "half"),
    (7, 600, 501, 501, 900, 449.5, 1.1, "rand"),     # mirror
    (15, 600, 501, 301, 900, 449.5, 1.0, "rand"),
    (31, 430, 411, 301, 600, 299.5, 0.8, "rand"),
    (4, 813, 811, 602, 1160, 579.5, 1.0, "half"),    # mirror with reflection
    (8, 613, 611, 501, 900, 449.0, 1.0, "half"),
    (15, 513, 511, 401, 727, 363.0, 1.0, "half"),
    (3, 800, 800, 600, 1140, 569.5, 1.0, "turn"),    # quarter turn
    (7, 800, 800, 400, 1140, 569.5, 1.0, "turn"),
    (15, 602, 602, 404, 860, 429.5, 1.0, "turn"),
    (9, 514, 514, 640, 740, 369.0, 1.0, "full"),     # two half-turn sets
    (4, 1030, 1030, 300, 1460, 729.5, 1.0, "half"),  # quarter turn, reflected set
    (8, 1030, 1030, 180, 1460, 729.5, 1.0, "half"),
    # items that fill one round of the device
    (64, 512, 500, 150, 729, 363.7, 1.0, "half"),      # plain, 64 columns
    (32, 700, 690, 101, 1000, 499.5, 1.0, "rand"),     # mirror, 64
    (16, 990, 1010, 81, 1440, 719.5, 1.0, "rand"),     # 32
    (16, 1020, 1010, 101, 1450, 724.5, 1.0, "half"),   # mirror with reflection, 64
    (32, 700, 700, 80, 1000, 499.5, 1.0, "turn"),      # quarter turn, 64
    (4, 1950, 1950, 100, 2780, 1389.5, 1.0, "half"),   # quarter turn with reflection, 32
    (8, 1400, 1400, 240, 1990, 994.5, 1.0, "half"),    # 64
])
def test_adjoint_by_columns(xct, case):
    """Every kind and column count of the matrix-core kernel."""
    S, nx, ny, na, nd, c, px, kind = case
    rng = np.random.default_rng(950 + S)
    if kind == "turn":  # arbitrary angles and the same a quarter turn on
        a = np.sort(rng.uniform(0.01, 0.5 * math.pi, na // 2))
        a = np.concatenate([a, a + 0.5 * math.pi])
    else:
        a = _angles(kind, na, rng)
    g = synth.Geometry(n_angles=na, n_det=nd, nx=nx, ny=ny, center=c, pixel_size=px, angles=a)
    q = rng.standard_normal((S, na, nd)) * np.linspace(0.5, 2.0, S)[:, None, None]
    say("adjoint by columns", case)
    img = xct.project_adjoint(to_dev(q), g)
    torch.cuda.synchronize()
    ref = oracle.backproject(q.astype(np.float32).astype(np.float64), g, oracle.adjoint_scale(g))
    for z in range(S):
        assert rel_l2(img[z].cpu().numpy(), ref[z]) < TOL, z


@pytest.mark.parametrize("case", [
    (61, 413, 390, 301, 600, 299.7),   # 64 columns, plain
    (4, 813, 811, 602, 1160, 579.5),   # 16 columns, mirror with reflection
    (4, 1030, 1030, 300, 1460, 729.5),  # 32 columns, quarter turn with reflection
])
def test_non_finite_rows_leave_the_matrix_cores(xct, case):
    """The slab takes vector kernels (not always xct_backproject's: slices in
    pairs): the same pixels stay finite, and lie within those kernels' gate."""
    S, nx, ny, na, nd, c = case
    g = synth.Geometry(n_angles=na, n_det=nd, nx=nx, ny=ny, center=c)
    say("non-finite", case)
    for bad in (float("nan"), float("-inf")):
        q = torch.randn(S, na, nd, generator=torch.Generator().manual_seed(5)).cuda()
        q[S - 1, na // 3, nd // 2] = bad
        img = xct.project_adjoint(q, g)
        want = torch.empty_like(img)
        xct.xct_backproject(g, q, want, 1.0)
        torch.cuda.synchronize()
        assert not torch.isfinite(img).all()
        assert torch.equal(torch.isfinite(img), torch.isfinite(want))
        ok = torch.isfinite(want)
        assert rel_l2(img[ok].cpu().numpy(), want[ok].cpu().double().numpy()) < TOL_VECTOR


@pytest.mark.parametrize("case", [0, 4, 7, 9])
def test_non_finite_samples_reach_the_same_pixels(xct, case):
    """A NaN and an infinity in the rows give non-finite pixels where the
    oracle's taps meet them and nowhere else."""
    S, nx, ny, na, nd, c, px, kind = CASES[case]
    rng = np.random.default_rng(40 + case)
    g = synth.Geometry(n_angles=na, n_det=nd, nx=nx, ny=ny, center=c, pixel_size=px, angles=_angles(kind, na, rng))
    q = rng.standard_normal((S, na, nd)).astype(np.float32)
    q[S // 2, na // 2, nd // 2] = np.nan
    q[0, 0, nd // 3] = np.inf
    img = xct.project_adjoint(to_dev(q), g).cpu().numpy()
    mark = np.zeros(q.shape)
    mark[~np.isfinite(q)] = 1.0
    hit = oracle.backproject(mark, g) > 0
    clear = oracle.backproject(mark, g) == 0
    # (a tap's weight within rounding of zero may or may not count)
    assert np.isfinite(img[clear]).mean() > 0.999
    assert not np.isfinite(img[hit]).any() or (~np.isfinite(img[hit])).mean() > 0.999
    assert (~np.isfinite(img)).any()


@pytest.mark.parametrize("storage", [torch.float32, torch.float16, torch.bfloat16])
def test_batch_of_split_and_matrix_slabs(xct, storage):
    """One batch holding split and matrix slabs: each image equals its own
    call's bit for bit, and the oracle; with a workspace that lacks the scratch
    behind the filtered rows the vector kernels give the same within rounding."""
    rng = np.random.default_rng(5)
    slabs, refs = [], []
    for S, nx, ny, na, nd, c, px, kind in (CASES[9], CASES[6], CASES[4], CASES[3]):
        g = synth.Geometry(n_angles=na, n_det=nd, nx=nx, ny=ny, center=c, pixel_size=px, angles=_angles(kind, na, rng))
        p = torch.as_tensor(rng.standard_normal((S, na, nd))).to(torch.float32).to(storage)
        slabs.append((g, p.cuda(), torch.empty((S, ny, nx), device="cuda")))
        refs.append(oracle.fbp(p.to(torch.float64).numpy(), g, "hann"))
    xct.xct_fbp_batch(slabs, "hann")
    for (g, p, img), ref in zip(slabs, refs):
        alone = torch.empty_like(img)
        xct.xct_fbp_batch([(g, p, alone)], "hann")
        torch.cuda.synchronize()
        assert torch.equal(alone, img)
        assert rel_l2(img.cpu().numpy(), ref) < 2e-5
    base = 256 + 4 * 1024 + sum((p.numel() * 4 + 255) // 256 * 256 for _, p, _ in slabs)
    assert xct.xct_fbp_workspace_bytes(slabs) > base
    again = [(g, p, torch.empty_like(img)) for g, p, img in slabs]
    xct.xct_fbp_batch(again, "hann", workspace=torch.empty(base, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    for (_, _, img), (_, _, b) in zip(slabs, again):
        assert rel_l2(b.cpu().numpy(), img.cpu().numpy().astype(np.float64)) < 2e-5


@pytest.mark.parametrize("case", [
    # slices, nx, ny, angles, bins, centre, angle set
    (1, 130, 97, 40, 190, 94.3, "half"),
    (2, 256, 256, 90, 367, 183.0, "half"),
    (3, 200, 64, 33, 301, 150.0, "rand"),    # four-slice form, walks of different lengths
    (5, 97, 131, 60, 170, 84.5, "full"),
    (16, 420, 400, 1500, 600, 297.7, "half"),  # more workgroups than the device holds
])
def test_split_forward_projection(xct, case):
    """Calls too small to fill the device, whose walks over the image are split."""
    S, nx, ny, na, nd, c, kind = case
    rng = np.random.default_rng(70 + na)
    g = synth.Geometry(n_angles=na, n_det=nd, nx=nx, ny=ny, center=c, angles=_angles(kind, na, rng))
    x = rng.standard_normal((S, ny, nx))
    y = rng.standard_normal((S, na, nd))
    dx, dy = to_dev(x), to_dev(y)
    say("split forward", case)
    p = xct.forward_project(dx, g)
    r = torch.empty_like(dy)
    xct.xct_forward_residual(g, dx, dy, r)
    torch.cuda.synchronize()
    ref = oracle.forward(x.astype(np.float32).astype(np.float64), g)
    assert rel_l2(p.cpu().numpy(), ref) < TOL
    assert rel_l2(r.cpu().numpy(), y.astype(np.float32) - ref) < TOL


@pytest.mark.parametrize("case", [
    # slices, side, angles, bins, centre, pixel: square slices whose quarter of
    # a uniform half turn is walked for four turned copies
    (1, 512, 48, 730, 361.7, 1.0),     # N_p / 4 a row of two copies, the fewest angles
    (2, 512, 50, 730, 364.5, 1.0),     # N_p / 2 odd
    (1, 515, 96, 733, 366.0, 1.0),     # odd side
    (3, 512, 432, 300, 149.5, 0.4),    # a group of three
    (1, 640, 98, 460, 229.1, 0.5),     # a small pixel: wide hats
])
def test_forward_projection_by_turned_copies(xct, case):
    """Against the oracle; and by each row of the last angles of the quarter,
    which two copies share, against a call under the same angles that are no
    uniform half turn (its last angle apart)."""
    S, n, na, nd, c, pixel = case
    rng = np.random.default_rng(90 + na)
    g = synth.Geometry(n_angles=na, n_det=nd, nx=n, ny=n, center=c, pixel_size=pixel)
    x = rng.standard_normal((S, n, n))
    y = rng.standard_normal((S, na, nd))
    dx, dy = to_dev(x), to_dev(y)
    say("turned copies", case)
    p = xct.forward_project(dx, g)
    r = torch.empty_like(dy)
    xct.xct_forward_residual(g, dx, dy, r, -0.5)
    acc = dy.clone()
    xct.xct_forward_project(g, dx, acc, -0.5, accumulate=True)
    ang = np.asarray(g.angles, dtype=np.float64).copy()
    ang[-1] += 1e-3
    other = xct.forward_project(dx, synth.Geometry(n_angles=na, n_det=nd, nx=n, ny=n, center=c, pixel_size=pixel,
                                                   angles=ang))
    torch.cuda.synchronize()
    assert torch.equal(r, acc)
    ref = oracle.forward(x.astype(np.float32).astype(np.float64), g)
    assert rel_l2(p.cpu().numpy(), ref) < TOL
    assert rel_l2(r.cpu().numpy(), y.astype(np.float32) - 0.5 * ref) < TOL
    for k in range(na - 1):
        assert rel_l2(p[:, k].cpu().numpy(), other[:, k].cpu().double().numpy()) < 2 * TOL, k


@pytest.mark.parametrize("case", [
    # slices, nx, ny, angles, bins, centre, pixel, angle set
    (2, 150, 100, 40, 220, 109.3, 1.0, "rand"),    # one pair
    (3, 200, 130, 200, 330, 164.7, 1.2, "half"),   # two pairs, the second half empty, split
    (5, 100, 300, 64, 430, 214.2, 1.5, "half"),    # three pairs, wide windows
    (4, 96, 96, 48, 200, 99.4, 2.0, "rand"),       # the widest windows that fit
    (3, 100, 300, 70, 430, 214.2, 1.7, "rand"),    # a pair and one, wide windows
    (3, 333, 190, 90, 400, 199.3, 0.9, "half"),    # ragged tiles
    (3, 60, 44, 21, 260, 129.3, 3.0, "half"),      # too wide for pairs: generic
])
def test_slices_in_pairs(xct, case):
    """Any geometry (axis off the half bins), two slices at a time."""
    S, nx, ny, na, nd, c, px, kind = case
    rng = np.random.default_rng(300 + na)
    g = synth.Geometry(n_angles=na, n_det=nd, nx=nx, ny=ny, center=c, pixel_size=px, angles=_angles(kind, na, rng))
    q = rng.standard_normal((S, na, nd)) * np.linspace(0.5, 2.0, S)[:, None, None]
    say("pairs", case)
    img = xct.project_adjoint(to_dev(q), g)
    torch.cuda.synchronize()
    ref = oracle.backproject(q.astype(np.float32).astype(np.float64), g, oracle.adjoint_scale(g))
    for z in range(S):
        assert rel_l2(img[z].cpu().numpy(), ref[z]) < TOL_VECTOR, z
