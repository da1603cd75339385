"""The density's copy of the occupied MOs, laid out on the device: numbers of
occupied MOs around its padding, occupied ones scattered among the MOs, nuclei
that change the order of the AO rows (from 1024 AOs on), and C that only the
device holds.  Tolerances as for the density: 1e-12 of the sum of terms in FP64,
2e-5 in the mixed modes (FP32 products)."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_ao_rows import system

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("occupied", [1, 127, 128, 129])
@pytest.mark.parametrize("mode", ["fp64", "mixed_f32", "mixed_bf16x3"])
@pytest.mark.parametrize("ao", [75, 1100])
def test_occupied_mos(occupied, mode, ao):
    import paper_2512_16677_amd as q
    rng = np.random.default_rng(occupied)
    s = system(ao, seed=ao)
    s.mo_coef = rng.normal(0.0, 0.1, size=(150, ao))
    s.elec_coord = np.ascontiguousarray(s.elec_coord[:, :40])
    occ = np.zeros(150)
    occ[rng.permutation(150)[:occupied]] = rng.uniform(0.5, 2.0, occupied)
    B, tol = (53, 1e-12) if mode == "fp64" else (24, 2e-5)
    ctx = q.Context.from_system(s, mode=mode, bits=B)
    for change in ("none", "nuclei", "parameters", "nuclei"):
        if change == "nuclei":
            s.nucl_coord = np.ascontiguousarray(s.nucl_coord[:, [1, 0, 2]])
            ctx.set_nucleus(s.nucl_coord)
        if change == "parameters":
            s.mo_coef = np.ascontiguousarray(s.mo_coef[::-1])
            ctx._set_params_device(torch.from_numpy(s.nucl_coord).cuda(), torch.from_numpy(s.mo_coef).cuda())
        rho = ctx.get_density(occ).cpu().numpy().reshape(-1)
        ref, ref_abs = oracle.density(s, occ, B=B, with_abs=True)
        assert np.max(np.abs(rho - ref) / np.maximum(ref_abs, 1e-30)) <= tol, change
    assert bool((ctx.get_density(np.zeros(150)) == 0.0).all())
    ctx.close()
