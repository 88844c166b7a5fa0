"""The learned preconditioner on more images than a launch has workgroups (2^22
tiles) and than it could have (2^24 workgroups of 256 threads): images of one
pixel, where M multiplies by one number, the oracle's, and of 1 x 2 pixels."""
import numpy as np
import pytest

from oracle import learned as ol
from tests.test_learned_tiles import params


@pytest.mark.gpu
@pytest.mark.parametrize("count,shape", [((1 << 22) + 5, (1, 2)), ((1 << 24) + 3, (1, 1))])
def test_apply_to_many_images(count, shape):
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    theta = ol.flatten(*params(5, 2))
    Ws, d = ol.unflatten(theta.astype(np.float32).astype(np.float64), 2, 16)
    n = shape[0] * shape[1]
    M = np.stack([ol.apply(Ws, d, e.reshape(1, *shape)).ravel() for e in np.eye(n)])   # M is symmetric
    net = sp.LearnedPrecond(2)
    net.set_params(theta)
    u = torch.randn(count, *shape, generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    got = net.apply(u)
    want = u.reshape(count, n).double() @ torch.from_numpy(M).cuda()
    err = (got.reshape(count, n).double() - want).norm() / want.norm()
    assert float(err) <= 1e-5
