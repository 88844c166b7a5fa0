"""Forms and launch shapes per geometry (geometry.cpp).

Host: tests/index_check/shape_check.cpp over the workload, ragged and random
geometries, geometries of axis-parallel angles alone, bin spacings down to the
smallest accepted and large images with few angles.

GPU, against the oracle at the operators' 1e-5 bar (f, a float64 sum of squares
of values the same to float64 rounding, to 1e-9): geometries of axis-parallel
angles alone, where a pixel meets up to four bins, and one geometry on each
side of every rule of R's parts, of either form; batched solves of them equal
single ones bit for bit."""
import math
import os
import subprocess

import numpy as np
import pytest

from oracle import projector as oproj
from oracle.geometry import Geometry as OG
from tests._problems import rel_l2
from tests.test_index_safety import geometries

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def build_checker(name, *flags):
    hipcc = "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = os.path.join(ROOT, "_build", name)
    os.makedirs(os.path.dirname(exe), exist_ok=True)
    subprocess.run([hipcc, "-std=c++17", "-ffp-contract=off", *flags, "-I", os.path.join(ROOT, "include"), "-o", exe,
                    os.path.join(ROOT, "tests", "index_check", "shape_check.cpp"),
                    os.path.join(ROOT, "paper_1807_10151_amd", "csrc", "geometry.cpp")],
                   check=True, capture_output=True, text=True)
    return exe


def lines(rows):
    return "\n".join(" ".join(repr(v) if isinstance(v, float) else str(v) for v in r) for r in rows) + "\n"


def test_shapes_of_every_geometry():
    exe = build_checker("shape_check", "-O1", "-g", "-Xarch_host", "-fsanitize=address", "-Xarch_host",
                        "-fsanitize=undefined", "-Xarch_host", "-fno-sanitize-recover=all")
    rows = [g[:9] for g in geometries()]
    rows += [(20, 30, a, 60, 1.0, t0, math.pi / 2, ds, 0.13) for a in (1, 2, 4) for t0 in (0.0, math.pi / 2)
             for ds in (0.375, 0.4, 0.5, 0.51, 0.9, 1.0, 1.7)]
    rows += [(50, 67, 61, 83, 1.0, 0.2, 0.05, ds, 0.3) for ds in (0.375, 0.5, 0.7, 0.94, 1.0, 1.2, 2.5)]
    rows += [(n, m, a, int(1.1 * max(n, m)), 1.0, 0.1, -1.0, ds, 0.3) for n, m in ((900, 900), (520, 510), (300, 1300))
             for a in (10, 60, 150, 300) for ds in (0.92, 1.0)]
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0", UBSAN_OPTIONS="halt_on_error=1")
    res = subprocess.run([exe], input=lines(rows), capture_output=True, text=True, env=env, timeout=600)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
    assert f"checked {len(rows)} geometries" in res.stdout


def test_set_up_evaluates_few_rays():
    exe = build_checker("shape_time", "-O2")
    rows = [(64, 64, 90, 91, 1.0, 0.0, -1.0, 1.0, 0.0), (243, 243, 360, 345, 0.0752, 0.0, -1.0, 0.0752, 0.0),
            (512, 512, 720, 725, 1.0, 0.0, -1.0, 1.0, 0.0), (300, 420, 200, 700, 1.0, 0.1, -1.0, 0.93, 0.3)]
    res = subprocess.run([exe, "time"], input=lines(rows), capture_output=True, text=True, timeout=600)
    print(res.stdout)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]


@pytest.mark.gpu
@pytest.mark.parametrize("n_angles,theta0", [(1, 0.0), (1, math.pi / 2), (2, 0.0), (4, 0.0)])
@pytest.mark.parametrize("ds,offset", [(0.375, 0.13), (0.4, 0.13), (0.5, 0.0), (0.5, 0.13), (0.9, 0.13), (1.0, 0.0), (2.5, 0.13)])
def test_axis_parallel_angles_alone(n_angles, theta0, ds, offset):
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    kw = {"theta0": theta0, "dtheta": math.pi / 2, "bin_spacing": ds, "bin_offset": offset}
    og, g = OG(33, 20, n_angles, 70, **kw), sp.Geometry(33, 20, n_angles, 70, **kw)
    rng = np.random.default_rng(n_angles)
    y = rng.standard_normal((n_angles, 70)).astype(np.float32)
    x = rng.standard_normal((33, 20)).astype(np.float32)
    R, RT = oproj.matrix(og, "closed")
    yt, xt = torch.from_numpy(y).cuda(), torch.from_numpy(x).cuda()
    y64, x64 = y.astype(np.float64).ravel(), x.astype(np.float64).ravel()
    assert rel_l2(sp.sp_project(g, xt).cpu().numpy(), R @ x64) <= 1e-5
    assert rel_l2(sp.sp_backproject(g, yt).cpu().numpy(), RT @ y64) <= 1e-5
    assert rel_l2(sp.sp_gradient(g, xt, yt)[0].cpu().numpy(), RT @ (R @ x64 - y64)) <= 1e-5


# on 8192 wave slots: one-ray parts (m: through memory) / two-ray parts
SHAPES = [
    (7, 700, 100, 48),      # 4 / 8
    (7, 700, 1800, 48),     # 4m / 8
    (7, 700, 3900, 48),     # 3m / 8
    (7, 700, 5600, 48),     # 2 / 8
    (256, 4, 1300, 60),     # 4 / 4
    (256, 4, 2700, 60),     # 2 / 2
    (256, 4, 7000, 60),     # 1 / 2
    (20, 24, 3000, 40),     # 4 / 4
    (20, 24, 6000, 40),     # 2 / 2
    (20, 24, 11000, 40),    # 1 / 2
    (40, 1100, 20, 1000),   # 8m / 8
]


@pytest.mark.gpu
@pytest.mark.parametrize("ds", [0.92, 1.0])
@pytest.mark.parametrize("rows,cols,n_angles,n_bins", SHAPES)
def test_parts_against_the_oracle(rows, cols, n_angles, n_bins, ds):
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    kw = {"bin_spacing": ds, "bin_offset": 0.13}
    og, g = OG(rows, cols, n_angles, n_bins, **kw), sp.Geometry(rows, cols, n_angles, n_bins, **kw)
    rng = np.random.default_rng(rows + n_angles)
    x = rng.standard_normal((rows, cols)).astype(np.float32)
    b = rng.standard_normal((n_angles, n_bins)).astype(np.float32)
    R, _ = oproj.matrix(og, "closed")
    want = R @ x.astype(np.float64).ravel()
    res = want - b.astype(np.float64).ravel()
    xt, bt = torch.from_numpy(x).cuda(), torch.from_numpy(b).cuda()
    assert rel_l2(sp.sp_project(g, xt).cpu().numpy(), want) <= 1e-5
    r, f = sp.sp_residual(g, xt, bt)
    assert rel_l2(r.cpu().numpy(), res) <= 1e-5
    assert abs(float(f) - float(res @ res)) <= 1e-9 * float(res @ res)


@pytest.mark.gpu
@pytest.mark.parametrize("rows,cols,n_angles,n_bins", [s for s in SHAPES if s[2] <= 4000])
def test_batched_equals_single(rows, cols, n_angles, n_bins):
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    gs = [sp.Geometry(rows, cols, n_angles, n_bins), sp.Geometry(24, 20, 30, 33)]
    rng = np.random.default_rng(n_angles)
    bs = [torch.from_numpy(rng.uniform(0, 10, (g.n_angles, g.n_bins)).astype(np.float32)).cuda() for g in gs]
    kw = dict(K=1, a=0.5, gamma=0.5, mu=1e-5, rho=0.8, max_iter=4)
    for g, b, got in zip(gs, bs, sp.sp_suppcg_solve_batched(gs, bs, **kw)):
        one = sp.sp_suppcg_solve(g, b, None, **kw)
        np.testing.assert_array_equal(got.x_half.cpu().numpy(), one.x_half.cpu().numpy())
        np.testing.assert_array_equal(got.x_last.cpu().numpy(), one.x_last.cpu().numpy())


@pytest.mark.gpu
@pytest.mark.parametrize("slices", [
    [(40, 37, 30, 59, 1.0), (48, 40, 30, 65, 0.9)],                              # 16 shares, a wave each; pixels
    [(300, 290, 20, 419, 1.0), (300, 300, 20, 426, 1.0), (33, 20, 30, 40, 0.9)],   # 16 shares in two turns; pixels
    [(420, 430, 24, 602, 1.0), (40, 37, 30, 59, 1.0)] * 4,                       # 8 shares and 16, grouped by XCD
    [(1441, 1473, 6, 2062, 1.0), (420, 430, 24, 602, 1.0), (20, 30, 9, 37, 1.0)],  # two tiles per wave and the others
])
def test_batched_backprojection_of_every_form(slices):
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    gs = [sp.Geometry(r, c, a, b, bin_spacing=ds) for r, c, a, b, ds in slices]
    rng = np.random.default_rng(len(slices))
    bs = [torch.from_numpy(rng.uniform(0, 10, (g.n_angles, g.n_bins)).astype(np.float32)).cuda() for g in gs]
    kw = dict(K=0, mu=1e-5, rho=0.8, max_iter=3)
    for g, b, got in zip(gs, bs, sp.sp_suppcg_solve_batched(gs, bs, **kw)):
        one = sp.sp_suppcg_solve(g, b, None, **kw)
        np.testing.assert_array_equal(got.x_half.cpu().numpy(), one.x_half.cpu().numpy())
        np.testing.assert_array_equal(got.x_last.cpu().numpy(), one.x_last.cpu().numpy())
