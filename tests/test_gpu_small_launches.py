"""Launch shapes of small calls: the shells of a nucleus dealt out to several
workgroups of 64 points (few points), and 256-point workgroups beyond, on both
sides of the rule's edges and with a point count that ends inside a wavefront;
values, density and all three gradients against the oracle (1e-12 on rows, 1e-11
of the absolute terms on gradients, as for the larger systems)."""
import numpy as np
import pytest

import oracle
import synth
from tests.helpers import component_errors, grad_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("walkers", [1, 6, 13, 128, 333])
@pytest.mark.parametrize("screen", [False, True])
def test_water_at_the_edges_of_the_shell_split(walkers, screen):
    import paper_2512_16677_amd as q
    s = synth.water_like(walkers=walkers)
    w = synth.adjoint_weights(s, seed=3)
    ctx = q.Context.from_system(s)
    ctx.set_screening(screen)
    mo = ctx.get_mo_vgl().cpu().numpy()
    err = component_errors(mo.reshape(-1, 5, s.mo_num), oracle.mo_vgl(s).reshape(-1, 5, s.mo_num))
    assert max(err.values()) <= 1e-12, err
    g = ctx.adjoint(torch.from_numpy(w).cuda())
    ref = oracle.adjoint(s, w)
    for k in ("d_coef", "d_elec", "d_nucl"):
        assert grad_err(g[k].cpu().numpy().reshape(ref[k].shape), ref[k], ref[k + "_abs"]) <= 1e-11, k
    only = ctx.adjoint(torch.from_numpy(w).cuda(), d_coef=False, d_elec=False)
    assert torch.equal(only["d_nucl"], g["d_nucl"])
    only = ctx.adjoint(torch.from_numpy(w).cuda(), d_nucl=False, d_coef=False)
    assert torch.equal(only["d_elec"], g["d_elec"])
    ctx.close()
