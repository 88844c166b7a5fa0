"""S_TV steps that take their own decision (several inner steps, images below 2^18
pixels): the trials' counts, l and the image of the batched solver, which decides
in a launch of its own, bit for bit, and the standalone operator against the
oracle's trace, also where steps need more trials than the first four and where
they run out of them."""
import numpy as np
import pytest

from oracle import suppcg as osup
from tests._problems import rel_l2


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(1, 1), (1, 9), (16, 16), (33, 47), (511, 513), (512, 512)])
@pytest.mark.parametrize("K", [2, 3, 7])
def test_single_equals_batched(shape, K):
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    g = sp.Geometry(*shape, 16, int(1.5 * max(shape)) + 2)
    b = torch.from_numpy(np.abs(np.random.default_rng(K).standard_normal((g.n_angles, g.n_bins))).astype(np.float32)).cuda()
    kw = dict(K=K, a=0.7, gamma=0.5, mu=1e-5, rho=0.8, max_iter=3)
    got = sp.sp_suppcg_solve_batched([g], [b], **kw)[0]
    one = sp.sp_suppcg_solve(g, b, None, **kw)
    np.testing.assert_array_equal(got.x_half.cpu().numpy(), one.x_half.cpu().numpy())
    assert list(got.trace["ell"]) == list(one.trace["ell"])


@pytest.mark.gpu
@pytest.mark.parametrize("gamma,max_trials", [(1.0, 100), (300.0, 100), (300.0, 3), (300.0, 6)])
def test_perturb_against_the_oracle(gamma, max_trials):
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    x = np.random.default_rng(9).standard_normal((29, 31)).astype(np.float32)
    p = osup.TVParams(5, 0.5, gamma, max_trials)
    want = osup.s_tv(x.astype(np.float64), 0, p)
    g = sp.Geometry(29, 31, 4, 45)
    y, ell, _, trials = sp.sp_tv_perturb(g, torch.from_numpy(x).cuda(), 0, 5, 0.5, gamma, max_trials)
    assert int(ell) == want.ell and [int(t) for t in trials] == list(want.trials)
    assert rel_l2(y.cpu().numpy(), x.astype(np.float64) + want.s) <= 1e-5
