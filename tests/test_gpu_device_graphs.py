"""Two autograd graphs on one context whose coefficients and nuclei live on the
device, backward in reverse order and again in forward order, on the default and
on a side stream: each graph gets the oracle's gradients of its own inputs, also
where the nuclei of the two give the AO rows different orders (1100 AOs).
Tolerance 1e-11 of the sum of terms, as for parameters on the host."""
import copy

import numpy as np
import pytest

import oracle
import synth
from tests.helpers import grad_err
from tests.test_gpu_ao_rows import system

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ao", [25, 1100])
@pytest.mark.parametrize("side", [False, True])
def test_two_graphs_with_parameters_on_the_device(ao, side):
    import paper_2512_16677_amd as q
    s = synth.water_like(walkers=3) if ao == 25 else system(ao)
    rng = np.random.default_rng(17)
    systems, leaves, outs = [], [], []
    ctx = q.Context.from_system(s)
    ctx.set_screening(ao > 1000)
    stream = torch.cuda.Stream() if side else torch.cuda.default_stream()
    axes = ([0, 1, 2], [1, 0, 2])
    for g in range(2):
        sg = copy.copy(s)
        sg.mo_coef = s.mo_coef + 0.1 * g * rng.normal(size=s.mo_coef.shape)
        sg.nucl_coord = np.ascontiguousarray(s.nucl_coord[:, axes[g]])
        sg.elec_coord = np.ascontiguousarray(s.elec_coord[:, :, axes[g]])
        systems.append(sg)
        leaves.append([torch.from_numpy(a.copy()).cuda().requires_grad_(True)
                       for a in (sg.mo_coef, sg.nucl_coord, sg.elec_coord)])
    ws = [synth.adjoint_weights(s, seed=60 + g) for g in range(2)]
    wd = [torch.from_numpy(w).cuda() for w in ws]
    refs = [oracle.adjoint_products(sg, w) for sg, w in zip(systems, ws)]
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for x in leaves:
            outs.append(q.mo_vgl(ctx, *x))
        for order in ((1, 0), (0, 1)):
            for g in order:
                got = torch.autograd.grad(outs[g], leaves[g], grad_outputs=wd[g].view_as(outs[g]), retain_graph=True)
                for k, x in zip(("d_coef", "d_nucl", "d_elec"), got):
                    ref = refs[g][k]
                    assert grad_err(x.cpu().numpy().reshape(ref.shape), ref, refs[g][k + "_abs"]) <= 1e-11, (order, g, k)
    ctx.close()
