"""GPU: what a refused stencil launch says."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ddml = pytest.importorskip("paper_1601_04587_amd.ddml")
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("prec", [ddml.FP64, ddml.MIXED_FP32])
def test_time_stencil_takes_every_tile_order_and_names_the_last(prec):
    L = (8, 4, 4, 4)
    ctx = ddml.Context(L, ddml.BC_ANTIPERIODIC)
    one = torch.eye(3, dtype=torch.complex128, device="cuda:0").expand(int(np.prod(L)), 4, 3, 3).contiguous()
    torch.cuda.synchronize()
    gid = ctx.set_gauge(one, 0.13, 1.0)
    last = 0
    while True:
        try:
            assert ctx.time_stencil(gid, -1, 2, prec, 1, order=last)[0] > 0
        except ddml.DDMLError as e:
            assert e.code == ddml.EINVAL and "order 0..%d " % (last - 1) in str(e)
            break
        last += 1
    assert last == 6
    ctx.close()
