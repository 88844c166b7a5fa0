"""A geometry whose workspace cannot be allocated is refused with SP_ERR_ALLOC and
leaves nothing behind: the context's next call on an earlier geometry builds its
tables again and gives the same results."""
import ctypes

import numpy as np
import pytest


@pytest.mark.gpu
def test_earlier_geometry_after_a_failed_allocation():
    torch = pytest.importorskip("torch")
    import paper_1807_10151_amd as sp
    from paper_1807_10151_amd import _lib as L
    ctx = sp.Context(0)
    g = sp.Geometry(48, 40, 30, 65)
    rng = np.random.default_rng(2)
    x = torch.from_numpy(rng.standard_normal((48, 40)).astype(np.float32)).cuda()
    b = torch.from_numpy(rng.uniform(0, 10, (30, 65)).astype(np.float32)).cuda()
    before = [sp.sp_project(g, x, ctx=ctx), *sp.sp_gradient(g, x, b, ctx=ctx)]
    torch.cuda.synchronize()
    # 8 parts of 1.8e9 rays in float64: 115 GB beside 22 GB of padded sinograms
    big = sp.Geometry(1500, 1500, 60000, 30000)
    y = torch.empty(60000, 30000, device="cuda")
    free, _ = torch.cuda.mem_get_info()
    hold = torch.empty(max(free - (80 << 30), 0), dtype=torch.uint8, device="cuda")   # 80 GB left
    try:
        xb = torch.empty(1500, 1500, device="cuda")
        gc = big.c()
        ctx._stream()
        rc = ctx.lib.sp_project(ctx.h, ctypes.byref(gc), ctypes.c_void_p(xb.data_ptr()), ctypes.c_void_p(y.data_ptr()))
        assert rc == L.SP_ERR_ALLOC
    finally:
        del hold, y
        torch.cuda.empty_cache()
    after = [sp.sp_project(g, x, ctx=ctx), *sp.sp_gradient(g, x, b, ctx=ctx)]
    for p, q in zip(before, after):
        np.testing.assert_array_equal(p.cpu().numpy(), q.cpu().numpy())
    ctx.close()
