"""GPU: the operator on canonical fields, its operator block and the boundary block
where their kernels can go wrong: boxes cut in every direction, rows and boxes that
fill no whole wavefront or tile, every number of columns, inputs that are also the
output, and contexts without room for the working copy of the links.

Tolerance 1e-13 of the largest value: a component of D psi adds some 400 FP64
products of order one, so rounding stays below 400 x 1.1e-16 of it.
"""
import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu

ddml = pytest.importorskip("paper_1601_04587_amd.ddml")
torch = pytest.importorskip("torch")

DEV = "cuda:0"
KAPPA, CSW, BETA = 0.1340, 1.769, 6.0
TOL = 1e-13
BCS = {"periodic": (ddml.BC_PERIODIC, 0), "antiperiodic": (ddml.BC_ANTIPERIODIC, 1), "open": (ddml.BC_OPEN, 2)}
# lattice, domain: whole lattice; time slab from an odd slice to the lattice's end;
# cut in every direction with uneven extents; rows of two sites; whole tiles and XCD regions
BOXES = [((4, 4, 4, 4), (0, 0, 0, 0), (4, 4, 4, 4)),
         ((8, 4, 6, 10), (3, 0, 0, 0), (7, 4, 6, 10)),
         ((8, 6, 6, 18), (0, 1, 2, 1), (6, 5, 6, 17)),
         ((6, 4, 4, 2), (2, 0, 0, 0), (6, 4, 4, 2)),
         ((8, 16, 16, 32), (0, 0, 0, 0), (4, 16, 16, 32))]


def _field(L):
    return inputs.heatbath(L, BETA, 11, 4) if np.prod(L) < 4000 else inputs.random_links(L, 11, 0.3)


def _noise(L, n, seed=3):
    r = np.random.default_rng(seed)
    shape = (n, int(np.prod(L)), 4, 3)
    return r.normal(size=shape) + 1j * r.normal(size=shape)


def _close(got, ref):
    assert np.abs(got - ref).max() <= TOL * np.abs(ref).max()


@pytest.mark.parametrize("bc", sorted(BCS))
@pytest.mark.parametrize("L,lo,hi", BOXES)
def test_operator_and_boundary_on_any_box(L, lo, hi, bc):
    U = _field(L)
    C = oracle.clover_term(U, L, CSW)
    ctx = ddml.Context(L, BCS[bc][0])
    gid = ctx.set_gauge(torch.from_numpy(U).to(DEV), KAPPA, CSW)
    dom = ctx.set_domain(lo, hi)
    psi = _noise(L, 12)
    ref = oracle.apply_D(U, L, KAPPA, psi, C=C, antiperiodic=BCS[bc][1], lo=lo, hi=hi)
    cut = oracle.apply_boundary(U, L, psi, lo, hi, antiperiodic=BCS[bc][1])
    inside = oracle.domain_mask(L, lo, hi)
    for n in (1, 2, 5, 7, 9, 10, 12):
        x = torch.from_numpy(np.ascontiguousarray(psi[:n])).to(DEV)
        out = torch.full_like(x, float("nan"))
        got = ctx.apply_Dw(gid, dom, x, out, n).cpu().numpy()
        _close(got, ref[:n])
        assert np.all(got[:, ~inside] == 0)
        out = torch.full_like(x, float("nan"))
        got = ctx.apply_boundary(gid, dom, x, out, n, -0.5).cpu().numpy()
        assert np.abs(got + 0.5 * cut[:n]).max() <= TOL * max(1.0, np.abs(cut).max())
        assert np.all(got[:, ~inside] == 0)
    ctx.apply_Dw(gid, dom, x, x, 12)   # the output may be the input
    _close(x.cpu().numpy(), ref)
    ctx.close()


@pytest.mark.parametrize("room", [False, True])
def test_operator_block_and_level1_without_room_for_the_working_copy(room):
    """The pool hands out whole 2 MiB blocks, so each buffer of this lattice is one: the field,
    the flag, the region, five operator arrays and the walks take nine."""
    L, lo, hi = (8, 4, 4, 4), (2, 0, 1, 0), (6, 4, 3, 4)
    U = _field(L)
    psi = _noise(L, 3)
    x = torch.from_numpy(psi).to(DEV)
    MiB = 1 << 20
    ctx = ddml.Context(L, ddml.BC_ANTIPERIODIC, hbm_budget=(64 if room else 16) * MiB)
    gid = ctx.set_gauge(torch.from_numpy(U).to(DEV), KAPPA, CSW)
    got = ctx.apply_Dw(gid, ctx.set_domain(lo, hi), x, torch.zeros_like(x), 3).cpu().numpy()
    _close(got, oracle.apply_D(U, L, KAPPA, psi, C=oracle.clover_term(U, L, CSW), lo=lo, hi=hi))
    ctx.close()
    ctx = ddml.Context(L, ddml.BC_ANTIPERIODIC, hbm_budget=(64 if room else 6) * MiB)
    gid = ctx.set_gauge(torch.from_numpy(U).to(DEV), KAPPA, CSW)
    new = ctx.level1_update(gid, 1, 6, BETA, 5, 3 + 7, 2, 1)
    got = ctx.get_gauge(new, np.zeros_like(U))
    ctx.close()
    ref = oracle.level1_update(U, L, BETA, 5, 7, 1, 6, 2, 1)
    assert np.abs(got - ref).max() <= 1e-11   # as the other level-1 tests: the sampler's functions amplify rounding


@pytest.mark.parametrize("t0,t1", [(0, 6), (0, 5), (5, 6), (2, 6)])
def test_level1_slabs_at_the_ends_of_the_lattice(t0, t1):
    L = (6, 4, 6, 10)
    U = _field(L)
    ctx = ddml.Context(L, ddml.BC_PERIODIC)
    gid = ctx.set_gauge(torch.from_numpy(U).to(DEV), KAPPA, CSW)
    got = ctx.get_gauge(ctx.level1_update(gid, t0, t1, BETA, 9, 3 + 1, 1, 2), np.zeros_like(U))
    ctx.close()
    assert np.abs(got - oracle.level1_update(U, L, BETA, 9, 1, t0, t1, 1, 2)).max() <= 1e-11
