"""R's two forms have part counts of their own in the launch-shape table: a count
stored for the solvers' form leaves that of a float32 image in two rays per lane
to its rule, and the other way round.

Which count a form used shows in the last bits of a float64 sum over the rays:
f of sp_residual for the two-ray form, a solve's f for the other.  The two-ray
form itself is checked against the oracle at every count (1e-5; f to 1e-9, a sum
of squares of values the same to float64 rounding)."""
import os

import numpy as np
import pytest

import paper_1807_10151_amd as sp
from oracle import projector as oproj
from oracle.geometry import Geometry as OG
from tests._problems import rel_l2


@pytest.fixture()
def clean():
    sp.tuning_clear()
    yield
    sp.tuning_clear()


def test_counts_are_stored_and_saved_per_form(clean, tmp_path):
    g, h = sp.Geometry(64, 64, 90, 91), sp.Geometry(37, 53, 45, 61)
    sp.tuning_set(g, 2, 4, parts32=5)
    sp.tuning_set(h, 8, 2)
    assert sp.tuning_parts32(g) == 5 and sp.tuning_parts32(h) == 0
    assert {(k.rows, p, x) for k, p, x in sp.tuning_list()} == {(64, 2, 4), (37, 8, 2)}
    path = os.path.join(tmp_path, "shapes.json")
    sp.tuning_save(path)
    sp.tuning_clear()
    assert sp.tuning_parts32(g) == 0
    sp.tuning_load(path)
    assert sp.tuning_parts32(g) == 5 and sp.tuning_parts32(h) == 0
    sp.tuning_set(g, 4, 4)
    assert sp.tuning_parts32(g) == 0


def test_files_without_the_second_count_load(clean, tmp_path):
    path = os.path.join(tmp_path, "shapes.json")
    with open(path, "w") as f:
        f.write('{"shapes": [{"rows": 64, "cols": 64, "n_angles": 90, "n_bins": 91, "pixel": 1.0, "theta0": 0.0, '
                '"dtheta": null, "bin_spacing": 1.0, "bin_offset": 0.0, "parts": 8, "px": 4}]}')
    sp.tuning_load(path)
    (g, parts, px), = sp.tuning_list()
    assert (parts, px) == (8, 4) and sp.tuning_parts32(g) == 0


@pytest.mark.parametrize("parts32", [-1, 9])
def test_rejects_bad_counts(clean, parts32):
    with pytest.raises(sp.SupPCGError):
        sp.tuning_set(sp.Geometry(16, 16, 8, 24), 1, 4, parts32=parts32)
    assert sp.tuning_list() == []


def f_of(torch, g, x, b):
    return float(sp.sp_residual(g, x, b)[1]), float(sp.sp_suppcg_solve(g, b, None, max_iter=1).trace["f_half"][0])


@pytest.mark.gpu
def test_a_count_applies_to_its_form(clean):
    torch = pytest.importorskip("torch")
    g = sp.Geometry(120, 130, 100, 178)
    rng = np.random.default_rng(8)
    x = torch.from_numpy(rng.standard_normal((120, 130)).astype(np.float32)).cuda()
    b = torch.from_numpy(rng.uniform(0, 10, (100, 178)).astype(np.float32)).cuda()
    f32, f64 = f_of(torch, g, x, b)
    sp.tuning_set(g, 8, 4)
    one = f_of(torch, g, x, b)
    assert one[0] == f32 and one[1] != f64
    sp.tuning_set(g, 4, 4, parts32=8)   # 4: the rule's count
    two = f_of(torch, g, x, b)
    assert two[0] != f32 and two[1] == f64
    sp.tune_shapes(g)
    (_, parts, _), = sp.tuning_list()
    sp.tuning_set(g, parts, 4, parts32=sp.tuning_parts32(g))
    tuned = f_of(torch, g, x, b)
    assert tuned[0] == f32 or sp.tuning_parts32(g) != 0


@pytest.mark.gpu
@pytest.mark.parametrize("parts32", [1, 2, 3, 4, 5, 8])
@pytest.mark.parametrize("rows,cols,n_angles,n_bins", [(1, 1, 5, 3), (40, 33, 25, 33), (33, 40, 27, 65), (1, 200, 31, 201)])
def test_two_ray_counts_against_the_oracle(clean, rows, cols, n_angles, n_bins, parts32):
    torch = pytest.importorskip("torch")
    g = sp.Geometry(rows, cols, n_angles, n_bins)
    rng = np.random.default_rng(rows * 1000 + cols)
    x = rng.standard_normal((rows, cols)).astype(np.float32)
    b = rng.standard_normal((n_angles, n_bins)).astype(np.float32)
    want = oproj.matrix(OG(rows, cols, n_angles, n_bins), "closed")[0] @ x.astype(np.float64).ravel()
    res = want - b.astype(np.float64).ravel()
    sp.tuning_set(g, 1, 4, parts32=parts32)
    got = sp.sp_project(g, torch.from_numpy(x).cuda()).cpu().numpy()
    r, f = sp.sp_residual(g, torch.from_numpy(x).cuda(), torch.from_numpy(b).cuda())
    assert rel_l2(got, want) <= 1e-5 and rel_l2(r.cpu().numpy(), res) <= 1e-5
    assert abs(float(f) - float(res @ res)) <= 1e-9 * float(res @ res)
