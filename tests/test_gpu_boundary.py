"""GPU: the boundary block by runs of 16 sites and by rows, on a field and on a version of it."""
import time

import numpy as np
import pytest

import inputs
import oracle

pytestmark = pytest.mark.gpu

ddml = pytest.importorskip("paper_1601_04587_amd.ddml")
torch = pytest.importorskip("torch")

DEV = "cuda:0"
KAPPA, CSW = 0.1340, 1.769
TOL = 1e-13   # at most eight hops of 12 products of order one in FP64 each


# rows of 2 and 6 sites (runs over several rows), one face in time only; long rows with
# their ends cut, of a whole and of an uneven number of 16-site passes, and not cut
@pytest.mark.parametrize("version", [False, True])
@pytest.mark.parametrize("L,lo,hi", [((4, 4, 2, 2), (1, 0, 0, 0), (3, 4, 2, 2)),
                                     ((6, 4, 4, 6), (2, 1, 1, 1), (6, 3, 3, 5)),
                                     ((4, 4, 2, 32), (0, 1, 0, 3), (2, 3, 2, 31)),
                                     ((4, 2, 4, 26), (1, 0, 1, 0), (3, 2, 3, 24)),
                                     ((4, 2, 4, 26), (2, 0, 0, 0), (4, 2, 2, 26))])
def test_boundary_block_of_a_field_and_of_a_version(L, lo, hi, version):
    U = inputs.random_links(L, 7, 0.3)
    V3 = int(np.prod(L[1:]))
    r = np.random.default_rng(4)
    shape = (12, int(np.prod(L)), 4, 3)
    psi = r.normal(size=shape) + 1j * r.normal(size=shape)
    ctx = ddml.Context(L, ddml.BC_ANTIPERIODIC)
    gid, dom = ctx.set_gauge(torch.from_numpy(U).to(DEV), KAPPA, CSW), ctx.set_domain(lo, hi)
    if version:   # other links on slices 1 and 2: one face of every domain has them
        U = np.concatenate([U[:V3], inputs.random_links(L, 8, 0.3)[V3:3 * V3], U[3 * V3:]])
        gid = ctx.set_gauge_region(gid, 1, 3, torch.from_numpy(np.ascontiguousarray(U[V3:3 * V3])).to(DEV))
    ref = oracle.apply_boundary(U, L, psi, lo, hi, antiperiodic=1)
    for n in (1, 5, 12):
        x = torch.from_numpy(np.ascontiguousarray(psi[:n])).to(DEV)
        got = ctx.apply_boundary(gid, dom, x, torch.full_like(x, float("nan")), n, 2.0).cpu().numpy()
        assert np.abs(got - 2.0 * ref[:n]).max() <= TOL * 2.0 * np.abs(ref).max()
        assert np.all(got[ref[:n] == 0] == 0)
    ctx.close()


def test_boundary_block_of_short_rows_takes_no_longer_than_of_long_rows():
    """The same number of sites, two slices of them with a face: the same bytes.  A third more is
    left for the index arithmetic."""
    def median(L):
        ctx = ddml.Context(L, ddml.BC_ANTIPERIODIC)
        gid = ctx.set_gauge(torch.from_numpy(inputs.random_links(L, 7, 0.3)).to(DEV), KAPPA, CSW)
        dom = ctx.set_domain((8, 0, 0, 0), (24,) + L[1:])
        x = torch.randn((12, int(np.prod(L)), 4, 3), dtype=torch.complex128, device=DEV)
        out = torch.zeros_like(x)
        times = []
        for _ in range(25):
            torch.cuda.synchronize()
            t = time.perf_counter()
            ctx.apply_boundary(gid, dom, x, out, 12)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t)
        ctx.close()
        return sorted(times)[12]

    short, long = median((32, 64, 32, 2)), median((32, 16, 8, 32))
    assert short <= 1.33 * long, (short, long)
