"""GPU: a column of a call does not depend on how many columns the call has.

The number of columns decides the workgroup of the staged stencil (one wave
per column, plus waves that only stage) and, in FP64, whether the operator data
are staged at all.  A column's arithmetic is the same in each, so every result
is compared bit for bit with the twelve-column call's.
"""
import numpy as np
import pytest

import inputs

pytestmark = pytest.mark.gpu

ddml = pytest.importorskip("paper_1601_04587_amd.ddml")
torch = pytest.importorskip("torch")

L = (8, 6, 4, 10)
KAPPA, CSW = 0.1340, 1.769


@pytest.fixture(scope="module")
def setup():
    ctx = ddml.Context(L, ddml.BC_ANTIPERIODIC)
    dev = torch.device("cuda:0")
    gid = ctx.set_gauge(torch.from_numpy(inputs.heatbath(L, 6.0, 77, 10)).to(dev), KAPPA, CSW)
    r = np.random.default_rng(5)
    V = int(np.prod(L))
    src = torch.from_numpy(r.normal(size=(12, V, 4, 3)) + 1j * r.normal(size=(12, V, 4, 3))).to(dev)
    # ragged: 6 * 6 * 4 * 10 / 2 = 720 sites of a parity, 11.25 tiles
    yield ctx, gid, ctx.set_domain((1, 0, 0, 0), (7,) + L[1:]), src
    ctx.close()


@pytest.mark.parametrize("nrhs", [1, 2, 7, 11])
@pytest.mark.parametrize("prec", [ddml.FP64, ddml.MIXED_FP32, ddml.MIXED_FP16])
def test_column_is_the_same_in_any_number_of_columns(setup, prec, nrhs):
    ctx, gid, dom, src = setup
    prm = ddml.solver_params(tol=1e-10, prec=prec)
    full, some = torch.zeros_like(src), torch.zeros_like(src[:nrhs])
    for call in (lambda x, out: ctx.apply_eo(gid, dom, x, out, x.shape[0], prec),
                 lambda x, out: ctx.solve_domain(gid, dom, x, out, x.shape[0], prm)):
        call(src, full)
        call(src[:nrhs].contiguous(), some)
        torch.cuda.synchronize()
        assert torch.equal(torch.view_as_real(some), torch.view_as_real(full[:nrhs]))
