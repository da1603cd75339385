"""Jastrow of every number of walkers around the eight XCDs that the product deals
them out to, with few tiles a walker and with more than 1024: the value of a walker
does not depend on the others (bit for bit, whatever XCD it runs on), and agrees
with the pairwise oracle within 1e-12 of the sum of absolute terms."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nn,ne,walkers", [(5, 20, range(1, 26)), (270, 610, (1, 3, 4, 6, 7, 8, 9, 14, 15))])
def test_numbers_of_walkers(nn, ne, walkers):
    import paper_2512_16677_amd as q
    nord, kappa = 5, 0.7
    rng = np.random.default_rng(nn)
    nucl = rng.uniform(-8.0, 8.0, size=(nn, 3))
    elec = nucl[rng.integers(nn, size=(max(walkers), ne))] + rng.normal(size=(max(walkers), ne, 3))
    c = rng.normal(scale=0.2, size=(q.jastrow_een_terms(nord), nn))
    check = elec[:25] if nn < 100 else elec[:1]
    ref = oracle.jastrow_een(check, nucl, kappa, nord, c)
    ref_abs = oracle.jastrow_een(check, nucl, kappa, nord, np.abs(c))
    ctx = q.Context()
    ctx.set_nucleus(nucl)
    ctx.set_tile("jastrow_p", 1)  # 16 x 16: the most tiles
    for n in sorted(walkers, reverse=True):
        ctx.set_point(np.ascontiguousarray(elec[:n]))
        j = ctx.jastrow_een(nord, kappa, c).cpu().numpy()
        if n == max(walkers):
            every = j
        m = min(n, len(ref))
        assert np.all(np.abs(j[:m] - ref[:m]) <= 1e-12 * ref_abs[:m]), n
        assert np.array_equal(j, every[:n]), n
    ctx.close()


def test_workspace_of_small_molecules():
    """Rows of two electrons and two nuclei are not padded to cache lines: the
    arrays of a walker hold about 130 doubles (800 in padded rows)."""
    import paper_2512_16677_amd as q
    n = 200000
    elec = np.random.default_rng(0).normal(size=(n, 2, 3))
    nucl = np.array([[0.0, 0.0, -0.7], [0.0, 0.0, 0.7]])
    c = np.ones((q.jastrow_een_terms(5), 2))
    ctx = q.Context()
    ctx.set_nucleus(nucl)
    ctx.set_point(elec)
    out = torch.empty(n, dtype=torch.float64, device="cuda")
    ctx.set_tile("jastrow_p", 0)
    ctx.det_adj(torch.eye(5, dtype=torch.float64, device="cuda"))  # the library is loaded
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    j = ctx.jastrow_een(5, 0.8, c, out=out)
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] <= 2048 * n
    ref = oracle.jastrow_een(elec[:50], nucl, 0.8, 5, c)
    assert np.all(np.abs(j.cpu().numpy()[:50] - ref) <= 1e-12 * oracle.jastrow_een(elec[:50], nucl, 0.8, 5, np.abs(c)))
    ctx.close()
