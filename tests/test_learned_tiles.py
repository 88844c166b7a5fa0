"""The learned preconditioner's convolutions at the edges of their tiles: images
narrower than a 16-pixel tile, one pixel more or less, strips of one row and of
the remainder, one image and many, one to three layers.  Against the
float64 oracle at the operators' 1e-5 bar."""
import numpy as np
import pytest

from oracle import learned as ol
from tests._problems import rel_l2


def params(seed, layers):
    rng = np.random.default_rng(seed)
    Ws = [rng.standard_normal((16, 1 if l == 0 else 16, 3, 3)) / 6 for l in range(layers)]
    return Ws, rng.standard_normal(16)


@pytest.mark.gpu
@pytest.mark.parametrize("layers", [1, 2, 3])
@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 1, 17), (1, 17, 1), (3, 2, 15), (1, 16, 16), (1, 33, 48), (40, 70, 31),
                                   (1, 515, 530)])
def test_apply(shape, layers):
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    Ws, d = params(shape[1] + layers, layers)
    theta = ol.flatten(Ws, d)
    Ws, d = ol.unflatten(theta.astype(np.float32).astype(np.float64), layers, 16)
    net = sp.LearnedPrecond(layers)
    net.set_params(theta)
    u = np.random.default_rng(3).standard_normal(shape).astype(np.float32)
    got = net.apply(torch.from_numpy(u).cuda()).cpu().numpy()
    assert rel_l2(got, ol.apply(Ws, d, u.astype(np.float64))) <= 1e-5
