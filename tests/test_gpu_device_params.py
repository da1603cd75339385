"""Parameters handed over on the device (the autograd function with CUDA
tensors): the same results, bit for bit, as through the host, in every mode and
at sizes around the padding of the coefficient copies; refused values leave the
context as it was; the host-side users of C (density) see the new values."""
import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def system(mo):
    s = synth.water_like(walkers=7)
    rng = np.random.default_rng(mo)
    s.mo_coef = rng.normal(0.0, 0.2, size=(mo, s.ao_num))
    return s


@pytest.mark.parametrize("mode", ["fp64", "mixed_f32", "mixed_bf16x3"])
@pytest.mark.parametrize("mo", [1, 31, 33, 128, 129])
def test_device_and_host_parameters_agree(mode, mo):
    import paper_2512_16677_amd as q
    s = system(mo)
    nucl = s.nucl_coord + 0.25
    w = torch.randn((7, s.elec_num, 5, mo), dtype=torch.float64, device="cuda")
    r = torch.from_numpy(np.ascontiguousarray(s.elec_coord)).cuda()
    got = []
    for dev in ("cpu", "cuda"):
        ctx = q.Context.from_system(s, mode=mode)
        ctx.get_mo_vgl()  # tables and copies of the first parameters
        C = torch.from_numpy(s.mo_coef[:, ::-1].copy()).to(dev).requires_grad_(True)
        R = torch.from_numpy(nucl.copy()).to(dev).requires_grad_(True)
        mo_t = q.mo_vgl(ctx, C, R, r)
        g = torch.autograd.grad(mo_t, (C, R), grad_outputs=w)
        rho = ctx.get_density(np.linspace(0.0, 2.0, mo) if mo > 1 else np.ones(1))
        got.append([mo_t.detach()] + [x.cpu() for x in g] + [rho])
        ctx.close()
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("bad", ["C", "R"])
def test_refused_device_parameters_leave_the_context(bad):
    import paper_2512_16677_amd as q
    s = system(33)
    ctx = q.Context.from_system(s, points_on_device=True)
    before = ctx.get_mo_vgl()
    C = torch.from_numpy(s.mo_coef + 1.0).cuda()
    R = torch.from_numpy(s.nucl_coord + 1.0).cuda()
    (C if bad == "C" else R).view(-1)[-1] = float("inf")
    with pytest.raises(q.QmkError) as e:
        q.mo_vgl(ctx, C, R, torch.from_numpy(np.ascontiguousarray(s.elec_coord)).cuda())
    assert e.value.status == q.QMK_NONFINITE
    ctx.set_point(torch.from_numpy(np.ascontiguousarray(s.elec_coord)).cuda())
    assert torch.equal(ctx.get_mo_vgl(), before)
    ctx.close()
