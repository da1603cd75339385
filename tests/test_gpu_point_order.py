"""The point order of the screened products on both sides of its table limits:
four rings of points per nucleus or one (4096 and 4097 nuclei; 1,100,000
points), histogram blocks of 256 points or 1024 (16,384 nuclei and 70,000
points).  Only exact zeros are skipped, so the screened result equals the dense
one; sampled rows match the oracle to 1e-12."""
import numpy as np
import pytest

import oracle
import synth
from tests.helpers import rownorm_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nuclei,points", [(4096, 300), (4097, 300), (16384, 70000), (1000, 1100000)])
def test_screened_equals_dense(nuclei, points):
    import paper_2512_16677_amd as q
    s = synth.water_like(walkers=1)
    rng = np.random.default_rng(nuclei)
    # the molecule's own nuclei carry the shells, the others only order points
    s.nucl_coord = np.concatenate([s.nucl_coord, rng.uniform(-4.0, 4.0, size=(nuclei - s.nucl_num, 3))])
    s.nucl_charge = np.ones(nuclei)
    s.mo_coef = s.mo_coef[:5].copy()
    s.elec_coord = rng.uniform(-4.0, 4.0, size=(1, points, 3))
    ctx = q.Context.from_system(s)
    dense = ctx.get_mo_vgl()
    ctx.set_screening(True)
    assert bool((ctx.get_mo_vgl() == dense).all())
    idx = np.unique(np.r_[0, points - 1, rng.integers(0, points, 200)])
    rows = dense.reshape(points, 5, s.mo_num)[torch.from_numpy(idx).cuda()].cpu().numpy()
    assert rownorm_err(rows, oracle.mo_vgl(s, points=s.points()[idx])).max() <= 1e-12
    ctx.close()
