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


@pytest.mark.gpu
@pytest.mark.parametrize("layers", [1, 2, 3])
@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 1, 17), (3, 17, 15), (2, 16, 33), (300, 20, 24)])
def test_loss_gradient(shape, layers):
    """The weight gradients' tiles: fewer pixels than a tile, one more, and more
    tiles than blocks (the bar of the existing gradient test, 1e-4)."""
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    Ws, d = params(shape[2] + layers, layers)
    theta = ol.flatten(Ws, d)
    Ws, d = ol.unflatten(theta.astype(np.float32).astype(np.float64), layers, 16)
    net = sp.LearnedPrecond(layers)
    net.set_params(theta)
    rng = np.random.default_rng(6)
    Av, v = (rng.standard_normal(shape).astype(np.float32) for _ in range(2))
    idx = np.arange(shape[0], dtype=np.int32)[::-1].copy()
    loss, gW, gd = ol.loss_and_grad(Ws, d, Av[idx].astype(np.float64), v[idx].astype(np.float64), margin=0)
    gl, gg = net.loss_grad(*(torch.from_numpy(a).cuda() for a in (Av, v, idx)), margin=0)
    assert abs(float(gl.item()) - loss) <= 1e-5 * abs(loss)
    got, off = gg.cpu().numpy().astype(np.float64), 0
    for part in [W.ravel() for W in gW] + [np.asarray(gd).ravel()]:
        assert rel_l2(got[off:off + part.size], part) <= 1e-4
        off += part.size
