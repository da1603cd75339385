"""Three-body Jastrow at the edges of the product's tiles and paddings (16
electrons, 16 nuclei, one more or fewer), for every order (each has its own
groups of powers) and every tile, against the pairwise oracle.  Tolerance: 1e-12
of the sum of absolute terms, as for the other Jastrow tests."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nn,ne", [(1, 2), (3, 15), (16, 16), (17, 33), (81, 31)])
@pytest.mark.parametrize("nord", [2, 3, 4, 5, 6, 7, 8])
def test_edges_of_tiles_and_paddings(nn, ne, nord):
    import paper_2512_16677_amd as q
    rng = np.random.default_rng(100 * nn + 10 * ne + nord)
    W, kappa = 3, 0.8
    nucl = rng.uniform(-4.0, 4.0, size=(nn, 3))
    elec = nucl[rng.integers(nn, size=(W, ne))] + rng.normal(size=(W, ne, 3))
    c = rng.normal(scale=0.2, size=(q.jastrow_een_terms(nord), nn))
    ref = oracle.jastrow_een(elec, nucl, kappa, nord, c)
    ref_abs = oracle.jastrow_een(elec, nucl, kappa, nord, np.abs(c))
    ctx = q.Context()
    ctx.set_nucleus(nucl)
    ctx.set_point(elec)
    for t in range(ctx.tile_count()):
        ctx.set_tile("jastrow_p", t)
        j = ctx.jastrow_een(nord, kappa, c).cpu().numpy()
        assert np.all(np.abs(j - ref) <= 1e-12 * ref_abs), t
    ctx.close()
