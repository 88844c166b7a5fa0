"""R^T over 2 x 2 pixel blocks.

Host: tests/index_check/quad_check.cpp compares every weight of the block form
with the chord length it stands for, over the workload, ragged and random
geometries and bin spacings on both sides of the rule that selects it.
Tolerance of a weight: the window index is a sum of three float64 terms of at
most a few thousand bins, so its fraction is off by about 1e-12 at most, and a
weight by that times the trapezoid's slope 1 / min(|cos|, |sin|).

GPU: sizes around the 16-pixel tiles, the share counts and the two-tile form,
float32 sinograms and the float64 residual, against the oracle at the 1e-5
bar of the operators, and 2 and 4 pixels per lane bit for bit."""
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


def test_block_weights_equal_chord_lengths():
    hipcc = "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = os.path.join(ROOT, "_build", "quad_check")
    os.makedirs(os.path.dirname(exe), exist_ok=True)
    subprocess.run([hipcc, "-std=c++17", "-O1", "-g", "-ffp-contract=off",
                    "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
                    "-Xarch_host", "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "include"), "-o", exe,
                    os.path.join(ROOT, "tests", "index_check", "quad_check.cpp"),
                    os.path.join(ROOT, "paper_1807_10151_amd", "csrc", "geometry.cpp")],
                   check=True, capture_output=True, text=True)
    rows = [(*g[:9], max(1, g[0] * g[1] * g[2] // 12_000_000)) for g in geometries()]
    rows += [(50, 67, 61, 83, 1.0, 0.2, 0.05, ds, 0.3, 1) for ds in (0.94, 0.95, 0.97, 1.0, 1.001, 1.2)]
    rows += [(19, 23, 40, 31, 1.0, t0, 2 * math.pi / 40, 1.0, 0.0, 1) for t0 in (0.0, 0.01, -1.3)]   # full turn
    text = "\n".join(" ".join(repr(v) if isinstance(v, float) else str(v) for v in r) for r in rows) + "\n"
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0", UBSAN_OPTIONS="halt_on_error=1")
    res = subprocess.run([exe], input=text, capture_output=True, text=True, env=env, timeout=600)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
    last = res.stdout.strip().splitlines()[-1].split()
    assert int(last[1]) == len(rows) and int(last[3]) >= 30


@pytest.mark.gpu
@pytest.mark.parametrize("rows,cols,n_angles,n_bins,kw", [
    (1, 1, 5, 3, {}), (2, 2, 6, 5, {}), (15, 17, 20, 25, {}), (16, 16, 24, 24, {}), (33, 31, 40, 47, {}),
    (417, 433, 24, 603, {}),               # 8 shares
    (1, 300, 31, 301, {}), (300, 1, 31, 301, {}),
    (48, 40, 64, 65, {"theta0": -1.3, "dtheta": 2 * math.pi / 64}),
    (48, 40, 30, 65, {"bin_spacing": 0.96}), (48, 40, 30, 65, {"bin_spacing": 1.2}),
    (48, 40, 30, 40, {"bin_offset": 9.5}),   # windows past the detector's ends
    (1441, 1473, 6, 2062, {}),             # two tiles per wave, 4 shares
])
def test_blocks_against_the_oracle(rows, cols, n_angles, n_bins, kw):
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    og = OG(rows, cols, n_angles, n_bins, **kw)
    g = sp.Geometry(rows, cols, n_angles, n_bins, **kw)
    rng = np.random.default_rng(rows * 1000 + cols)
    y = rng.standard_normal((n_angles, n_bins)).astype(np.float32)
    x = rng.standard_normal((rows, cols)).astype(np.float32)
    R, RT = oproj.matrix(og, "closed")
    yt, xt = torch.from_numpy(y).cuda(), torch.from_numpy(x).cuda()
    want = RT @ y.astype(np.float64).ravel()
    want_g = RT @ (R @ x.astype(np.float64).ravel() - y.astype(np.float64).ravel())
    got = {}
    for px in (4, 2):
        sp.tuning_set(g, 1, px)
        try:
            got[px] = (sp.sp_backproject(g, yt).cpu().numpy(), sp.sp_gradient(g, xt, yt)[0].cpu().numpy())
        finally:
            sp.tuning_set(g, 0, 0)
    assert rel_l2(got[4][0], want) <= 1e-5 and rel_l2(got[4][1], want_g) <= 1e-5
    assert np.array_equal(got[4][0], got[2][0]) and np.array_equal(got[4][1], got[2][1])
