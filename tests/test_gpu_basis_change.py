"""A context whose basis is replaced by a smaller one that pads to the same
number of rows: the AO arrays keep nothing of the rows that are gone, not even
where their values overflowed.  Oracle and tolerances as for a fresh context."""
import numpy as np
import pytest

import oracle
import synth
from tests.helpers import component_errors, rownorm_err
from tests.test_gpu_mixed import TOL

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def s_shells(n):
    """n normalised s shells of one primitive on the three nuclei of water."""
    s = synth.water_like(walkers=5)
    rng = np.random.default_rng(n)
    s.shell_nucleus, s.shell_ang_mom = np.sort(rng.integers(0, 3, n)), np.zeros(n, int)
    s.shell_prim_offset, s.exponent, s.coefficient = np.arange(n + 1), 10.0 ** rng.uniform(-1, 1, n), np.ones(n)
    s.mo_coef = rng.normal(0.0, 0.3, size=(9, n))
    return s


@pytest.mark.parametrize("mode", ["fp64", "mixed_f32", "mixed_bf16x3"])
@pytest.mark.parametrize("screening", [False, True])
@pytest.mark.parametrize("ao", [97, 100, 127])
def test_rows_of_a_larger_basis_are_cleared(mode, screening, ao):
    import paper_2512_16677_amd as q
    B = 53 if mode == "fp64" else 24
    big, s = s_shells(128), s_shells(ao)
    occ = np.linspace(0.5, 2.0, 9)
    ctx = q.Context.from_system(big, mode=mode, bits=B)
    ctx.set_screening(screening)
    n = np.ones(128)
    ctx.set_basis(big.shell_nucleus, big.shell_ang_mom, big.shell_prim_offset, big.exponent, 1e300 * n,
                  prim_factor=1e300 * n, shell_factor=n)  # finite inputs, infinite AOs
    ctx.set_mo_coef(big.mo_coef)
    for f in (ctx.get_mo_vgl, ctx.get_mo_value, lambda: ctx.get_density(occ)):
        assert not bool(torch.isfinite(f()).all())
    ctx.set_point(s.elec_coord + 0.25)
    ctx.get_mo_value()  # the value-only array holds such rows too
    ctx.set_point(s.elec_coord)
    ctx.set_basis(s.shell_nucleus, s.shell_ang_mom, s.shell_prim_offset, s.exponent, s.coefficient)
    ctx.set_mo_coef(s.mo_coef)
    tol = 1e-12 if mode == "fp64" else 2e-5  # value and density products are FP32 in the mixed modes
    v = ctx.get_mo_value().cpu().numpy().reshape(-1, 9)
    assert rownorm_err(v, oracle.mo_value(s, B=B)).max() <= tol
    rho = ctx.get_density(occ).cpu().numpy().reshape(-1)
    ref, ref_abs = oracle.density(s, occ, B=B, with_abs=True)
    assert np.max(np.abs(rho - ref) / ref_abs) <= tol
    e = component_errors(ctx.get_mo_vgl().cpu().numpy().reshape(-1, 5, 9), oracle.mo_vgl(s, B=B))
    if mode == "fp64":
        assert max(e.values()) <= 1e-12, e
    else:
        assert all(e[k] <= TOL[mode][k] for k in ("value", "gradient", "laplacian")), e
    ctx.close()
