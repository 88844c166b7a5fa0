"""M over the transform lengths P = 2 .. 4096 (each last pass, transforms per
thread and per workgroup, odd rows, images narrower than their length), single
and in a batch with other lengths, against the oracle.

The result is a float64 one rounded to float32 once: relative to the largest
error 2^-24 of an element, 1e-7 leaves the float64 transforms 4e-8."""
import numpy as np
import pytest

from oracle import precond as oprecond
from tests._problems import rel_l2

SIZES = [(1, 1), (2, 1), (1, 2), (3, 4), (4, 3), (5, 8), (9, 16), (16, 17), (33, 31), (64, 64), (65, 3), (2, 129),
         (256, 255), (257, 300), (512, 37), (513, 1024), (1, 1025), (2048, 5), (1100, 2048)]


@pytest.mark.gpu
@pytest.mark.parametrize("rows,cols", SIZES)
@pytest.mark.parametrize("mu,rho", [(1e-5, 0.8), (1e-3, 0.6)])
def test_precond_against_the_oracle(rows, cols, mu, rho):
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    g = np.random.default_rng(rows * 4099 + cols).standard_normal((rows, cols)).astype(np.float32)
    want = oprecond.apply(g.astype(np.float64), mu, rho)
    geom = sp.Geometry(rows, cols, 4, 5)
    x = torch.from_numpy(g).cuda()
    assert rel_l2(sp.sp_precond_apply(geom, x, mu, rho).cpu().numpy(), want) <= 1e-7
    sp.sp_precond_apply(geom, x, mu, rho, z=x)   # in place
    assert rel_l2(x.cpu().numpy(), want) <= 1e-7


@pytest.mark.gpu
@pytest.mark.parametrize("sizes", [[(1, 1), (3, 4), (33, 31)], [(5, 8), (64, 64), (257, 300), (2, 129)],
                                   [(1100, 9), (16, 17), (513, 40), (1, 2)]])
def test_batch_of_lengths_equals_single(sizes):
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    geoms = [sp.Geometry(r, c, 12, int(1.5 * max(r, c)) + 2) for r, c in sizes]
    rng = np.random.default_rng(3)
    bs = [torch.from_numpy(np.abs(rng.standard_normal((g.n_angles, g.n_bins))).astype(np.float32)).cuda() for g in geoms]
    kw = dict(K=2, a=0.5, gamma=0.5, mu=1e-5, rho=0.8, max_iter=3)
    got = sp.sp_suppcg_solve_batched(geoms, bs, **kw)
    for r, g, b in zip(got, geoms, bs):
        s = sp.sp_suppcg_solve(g, b, None, **kw)
        np.testing.assert_array_equal(r.x_half.cpu().numpy(), s.x_half.cpu().numpy())
        np.testing.assert_array_equal(r.trace["f_half"], s.trace["f_half"])
