"""R's two-ray form (a float32 image, two neighbouring rays per lane).

Host: tests/index_check/pair_check.cpp replays the wave table, the step ranges,
the gathered pixels and the path-length shares of both rays against clipping
each ray band by band, over the workload, ragged and random geometries and
bin spacings on both sides of the rule that selects the form.

GPU: wave tails, odd bin counts, part counts (1 to 8: in the workgroup and by
the combining launch) and the spacing rule's edges against the oracle, at the
operators' 1e-5 bar; the residual's f, a float64 sum of squares of values the
same to float64 rounding, to 1e-9.  The non-unit spacings carry an offset: at
one, whether an axis-parallel ray lies exactly on a pixel edge (and takes half
of each pixel) depends on how its position rounds."""
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


def test_pairs_cover_and_split_every_ray():
    hipcc = "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = os.path.join(ROOT, "_build", "pair_check")
    os.makedirs(os.path.dirname(exe), exist_ok=True)
    subprocess.run([hipcc, "-std=c++17", "-O1", "-g", "-ffp-contract=off",
                    "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
                    "-Xarch_host", "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "include"), "-o", exe,
                    os.path.join(ROOT, "tests", "index_check", "pair_check.cpp"),
                    os.path.join(ROOT, "paper_1807_10151_amd", "csrc", "geometry.cpp")],
                   check=True, capture_output=True, text=True)
    rows = [(*g[:9], max(1, g[2] * g[3] * max(g[0], g[1]) // 12_000_000)) for g in geometries()]
    rows += [(50, 67, 61, 83, 1.0, 0.2, 0.05, ds, 0.3, 1) for ds in (0.97, 1.0, 1.001, 1.2, 1.41, 1.42)]
    rows += [(19, 23, 40, 31, 1.0, t0, 2 * math.pi / 40, 1.0, 0.0, 1) for t0 in (0.0, 0.01, -1.3)]   # full turn
    text = "\n".join(" ".join(repr(v) if isinstance(v, float) else str(v) for v in r) for r in rows) + "\n"
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0", UBSAN_OPTIONS="halt_on_error=1")
    res = subprocess.run([exe], input=text, capture_output=True, text=True, env=env, timeout=600)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
    last = res.stdout.strip().splitlines()[-1].split()
    assert int(last[1]) == len(rows) and int(last[3]) >= 40


@pytest.mark.gpu
@pytest.mark.parametrize("parts", [0, 1, 2, 3, 4, 5, 8])
@pytest.mark.parametrize("rows,cols,n_angles,n_bins,kw", [
    (1, 1, 5, 3, {}), (3, 2, 7, 1, {}), (40, 33, 24, 32, {}), (40, 33, 25, 33, {}), (33, 40, 27, 65, {}),
    (1, 200, 31, 201, {}), (200, 1, 31, 201, {}),
    (48, 40, 64, 65, {"theta0": -1.3, "dtheta": 2 * math.pi / 64}),
    (48, 40, 30, 65, {"bin_spacing": 0.99, "bin_offset": 0.37}), (48, 40, 30, 45, {"bin_spacing": 1.4, "bin_offset": 0.37}),
    (48, 40, 30, 45, {"bin_spacing": 1.43, "bin_offset": 0.37}),
])
def test_pairs_against_the_oracle(rows, cols, n_angles, n_bins, kw, parts):
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    og = OG(rows, cols, n_angles, n_bins, **kw)
    g = sp.Geometry(rows, cols, n_angles, n_bins, **kw)
    rng = np.random.default_rng(rows * 1000 + cols)
    x = rng.standard_normal((rows, cols)).astype(np.float32)
    b = rng.standard_normal((n_angles, n_bins)).astype(np.float32)
    R, _ = oproj.matrix(og, "closed")
    want = R @ x.astype(np.float64).ravel()
    res = want - b.astype(np.float64).ravel()
    if parts:
        sp.tuning_set(g, parts, 4)
    try:
        got = sp.sp_project(g, torch.from_numpy(x).cuda()).cpu().numpy()
        r, f = sp.sp_residual(g, torch.from_numpy(x).cuda(), torch.from_numpy(b).cuda())
    finally:
        sp.tuning_set(g, 0, 0)
    assert rel_l2(got, want) <= 1e-5 and rel_l2(r.cpu().numpy(), res) <= 1e-5
    assert abs(float(f) - float(res @ res)) <= 1e-9 * float(res @ res)


@pytest.mark.gpu
def test_form_changes_on_one_context():
    """The same padded layout in either form, one after the other: the copies of
    the form that comes second are zeroed at their pads too."""
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    ctx = sp.Context(0)
    x = np.random.default_rng(5).standard_normal((48, 40)).astype(np.float32)
    for ds in (0.99, 1.2, 0.99, 1.0):
        kw = {"bin_spacing": ds, "bin_offset": 0.37}
        want = oproj.matrix(OG(48, 40, 30, 65, **kw), "closed")[0] @ x.astype(np.float64).ravel()
        got = sp.sp_project(sp.Geometry(48, 40, 30, 65, **kw), torch.from_numpy(x).cuda(), ctx=ctx)
        assert rel_l2(got.cpu().numpy(), want) <= 1e-5
