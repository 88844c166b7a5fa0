"""S_TV's decisions on either side of the size up to which an inner step takes its
own (2^16 pixels), with the first trials accepted, with more than the first four
needed, and with none accepted: TV values, l and images bit for bit those of the
batched solver, which decides in a launch of its own, the trial counts of every
step those of the oracle; and steps that try every trial in a row take no longer
than as many calls of one step, which never decide for themselves."""
import numpy as np
import pytest

from oracle import suppcg as osup
from tests._problems import rel_l2

SHAPES = [(200, 150), (256, 256), (257, 256), (300, 310)]
STEPS = [(0.5, 0.7, 100), (4e3, 0.5, 100), (1e6, 0.99999, 6), (1e6, 0.99999, 9)]   # gamma, a, max_trials


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("gamma,a,max_trials", STEPS)
def test_decisions_of_the_batched_solver(shape, gamma, a, max_trials):
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    g = sp.Geometry(*shape, 16, int(1.5 * max(shape)) + 2)
    b = torch.from_numpy(np.abs(np.random.default_rng(2).standard_normal((g.n_angles, g.n_bins))).astype(np.float32)).cuda()
    kw = dict(K=3, a=a, gamma=gamma, mu=1e-5, rho=0.8, max_iter=3, max_trials=max_trials)
    got = sp.sp_suppcg_solve_batched([g], [b], **kw)[0]
    one = sp.sp_suppcg_solve(g, b, None, **kw)
    np.testing.assert_array_equal(got.x_half.cpu().numpy(), one.x_half.cpu().numpy())
    for key in ("tv_half", "ell"):
        np.testing.assert_array_equal(np.asarray(got.trace[key]), np.asarray(one.trace[key]))


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("gamma,a,max_trials", STEPS)
def test_trials_of_the_oracle(shape, gamma, a, max_trials):
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    x = np.random.default_rng(9).standard_normal(shape).astype(np.float32)
    want = osup.s_tv(x.astype(np.float64), 0, osup.TVParams(4, a, gamma, max_trials))
    g = sp.Geometry(*shape, 4, 2 * max(shape))
    y, ell, _, trials = sp.sp_tv_perturb(g, torch.from_numpy(x).cuda(), 0, 4, a, gamma, max_trials)
    assert int(ell) == want.ell and [int(t) for t in trials] == list(want.trials)
    assert (max(want.trials) > 4) == (gamma > 1.0)
    assert rel_l2(y.cpu().numpy(), x.astype(np.float64) + want.s) <= 1e-5


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(240, 250), (440, 440)])
def test_rejected_trials_take_no_longer_in_a_row(shape):
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    x = torch.from_numpy(np.random.default_rng(1).standard_normal(shape).astype(np.float32)).cuda()
    g = sp.Geometry(*shape, 4, 2 * max(shape))

    def ms(K):
        best = 1e30
        for _ in range(4):
            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            e0.record()
            sp.sp_tv_perturb(g, x, 0, K, 0.99999, 1e6, 40)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1))
        return best

    assert ms(5) <= 1.4 * 5 * ms(1)
