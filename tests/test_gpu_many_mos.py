"""More MOs than 65,535 tiles of 32 columns of the coefficient copies."""
import numpy as np
import pytest

import oracle
import synth
from tests.helpers import component_errors

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_two_million_mos():
    import paper_2512_16677_amd as q
    n = 65536 * 32 + 1
    s = synth.tiny_system([0, 1], walkers=1)
    s.mo_coef = np.random.default_rng(3).normal(size=(n, s.ao_num))
    s.elec_coord = np.ascontiguousarray(s.elec_coord[:, :1])
    ctx = q.Context.from_system(s)
    got = ctx.get_mo_vgl().cpu().numpy().reshape(-1, 5, n)
    ctx.close()
    e = component_errors(got, oracle.mo_vgl(s))
    assert max(e.values()) <= 1e-12, e
