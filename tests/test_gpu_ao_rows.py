"""Systems of 1024 AOs and more, whose AO arrays keep their rows in an order of
their own (shells by reach and place): every result against the oracle and in
the caller's order, before and after the nuclei move, just below and just above
the size where the order changes.  Tolerances: FP64 1e-12 row-normwise as for
every size, BF16x3 the bounds stated for the mode (an operand's two planes leave
2^-17 of each term), its density (FP32 products) 2e-5."""
import numpy as np
import pytest

import oracle
import synth
from tests.helpers import component_errors, grad_err, rownorm_err
from tests.test_gpu_mixed import TOL

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def system(ao, seed=0):
    """ao AOs: d, s, p and f shells in turn, two primitives each, 40 nuclei in a long box."""
    rng = np.random.default_rng(seed)
    nn, ang, nuc, off, expo, coef = 40, [], [], [0], [], []
    left = ao
    while left:
        l = [2, 0, 1, 3][len(ang) % 4]
        while (l + 1) * (l + 2) // 2 > left:
            l -= 1
        ang.append(l)
        g = 10.0 ** rng.uniform(-1.0, 2.5)
        expo += [4.0 * g, g]
        coef += list(rng.uniform(0.2, 1.0, 2))
        off.append(len(expo))
        left -= (l + 1) * (l + 2) // 2
    nuc = np.sort(rng.integers(0, nn, size=len(ang)))
    base = synth.water_like(walkers=2)
    xyz = rng.uniform(0.0, 1.0, size=(nn, 3)) * [60.0, 8.0, 8.0]
    elec = (xyz[rng.integers(0, nn, size=(2, 150))] + rng.normal(size=(2, 150, 3)))
    s = type(base)(**{**base.__dict__, "nucl_charge": np.ones(nn), "nucl_coord": xyz,
                      "shell_nucleus": nuc, "shell_ang_mom": np.array(ang), "shell_prim_offset": np.array(off),
                      "exponent": np.array(expo), "coefficient": np.array(coef),
                      "mo_coef": rng.normal(0.0, 0.1, size=(37, ao)), "elec_coord": elec})
    return s


@pytest.mark.parametrize("ao", [1023, 1024, 1025, 2111])
@pytest.mark.parametrize("mode", ["fp64", "mixed_bf16x3"])
def test_every_result_at_and_around_the_threshold(ao, mode):
    import paper_2512_16677_amd as q
    s = system(ao, seed=ao)
    assert s.ao_num == ao
    fp64 = mode == "fp64"
    B = 53 if fp64 else 24
    tol = 1e-12 if fp64 else 2e-5
    tol_mo = 1e-12 if fp64 else TOL[mode]["value"]
    ctx = q.Context.from_system(s, mode=mode, bits=B)
    occ = np.linspace(0.5, 2.0, s.mo_num)
    w = synth.adjoint_weights(s, seed=5)
    wd = torch.from_numpy(w).cuda()
    for moved in (False, True):
        if moved:  # the curve through the nuclei, and with it the rows, changes
            s.nucl_coord = np.ascontiguousarray(s.nucl_coord[:, [1, 0, 2]])
            s.elec_coord = np.ascontiguousarray(s.elec_coord[:, :, [1, 0, 2]])
            ctx.set_nucleus(s.nucl_coord)
            ctx.set_point(s.elec_coord)
        a = ctx.get_ao_vgl().cpu().numpy().reshape(-1, 5, ao)  # the first build of the tables
        if fp64:
            assert rownorm_err(a, oracle.ao_vgl(s, B=B)).max() <= tol
        rho = ctx.get_density(occ).cpu().numpy().reshape(-1)
        ref, ref_abs = oracle.density(s, occ, B=B, with_abs=True)
        assert np.max(np.abs(rho - ref) / ref_abs) <= tol
        dense = ctx.get_mo_vgl()
        e = component_errors(dense.cpu().numpy().reshape(-1, 5, s.mo_num), oracle.mo_vgl(s, B=B))
        assert max(e.values()) <= tol_mo, e
        v = ctx.get_mo_value().cpu().numpy().reshape(-1, s.mo_num)
        assert rownorm_err(v, oracle.mo_value(s, B=B)).max() <= tol
        r = oracle.adjoint_products(s, w, B=B)
        for screening in (False, True):
            ctx.set_screening(screening)
            assert bool((ctx.get_mo_vgl() == dense).all())
            g = ctx.adjoint(wd)
            for k in ("d_coef", "d_elec", "d_nucl"):
                err = grad_err(g[k].cpu().numpy().reshape(r[k].shape), r[k], r[k + "_abs"])
                assert err <= (1e-11 if fp64 else TOL[mode]["grad"]), (k, err)
        ctx.set_screening(False)
    if fp64:
        d = np.linalg.norm(s.nucl_coord[:, None] - s.nucl_coord[None], axis=-1) + 9.0 * np.eye(s.nucl_num)
        z, rc = s.nucl_charge.astype(np.float64), np.minimum(0.5, 0.4 * d.min(axis=1))  # spheres apart
        ctx.set_mo_cusp(z, rc)
        got = ctx.get_mo_vgl().cpu().numpy().reshape(-1, 5, s.mo_num)
        e = component_errors(got, oracle.mo_vgl_cusp(s, z, rc))
        assert max(e.values()) <= tol, e
    ctx.close()


@pytest.mark.parametrize("swap", [False, True])
def test_device_parameters_and_batch(swap):
    import paper_2512_16677_amd as q
    s = system(1025, seed=1)
    w = torch.from_numpy(synth.adjoint_weights(s, seed=6)).cuda()
    r = torch.from_numpy(s.elec_coord).cuda()
    axes = [1, 0, 2] if swap else [0, 1, 2]  # another order of rows, or the same
    got = []
    for dev in ("cpu", "cuda"):
        ctx = q.Context.from_system(s)
        ctx.get_mo_vgl()
        C = torch.from_numpy(s.mo_coef[:, ::-1].copy()).to(dev).requires_grad_(True)
        R = torch.from_numpy(s.nucl_coord[:, axes].copy()).to(dev).requires_grad_(True)
        mo = q.mo_vgl(ctx, C, R, r)
        got.append([mo.detach().cpu()] + [g.cpu() for g in torch.autograd.grad(mo, (C, R), grad_outputs=w)])
        ctx.close()
    for a, b in zip(*got):
        assert torch.equal(a, b)
    mols = [s, synth.water_like(walkers=3)]
    ctxs = [q.Context.from_system(m, points_on_device=True) for m in mols]
    b = q.Batch(ctxs)
    ws = [torch.from_numpy(synth.adjoint_weights(m, seed=7)).cuda() for m in mols]
    b.run(ws=ws)  # tiles timed, graph captured
    outs, grads = b.run(ws=ws)
    torch.cuda.synchronize()
    for m, c, o, g, wi in zip(mols, ctxs, outs, grads, ws):
        assert rownorm_err(o.cpu().numpy().reshape(-1, 5, m.mo_num), oracle.mo_vgl(m)).max() <= 1e-12
        ref = oracle.adjoint_products(m, wi.cpu().numpy())
        for k in ("d_coef", "d_elec", "d_nucl"):
            assert grad_err(g[k].cpu().numpy().reshape(ref[k].shape), ref[k], ref[k + "_abs"]) <= 1e-11, k
    b.close()


@pytest.mark.parametrize("shells", [63, 64, 65, 128, 129, 200])
def test_screened_store_with_many_shells_on_a_nucleus(shells):
    """The screened AO store finds a group's shells to store 64 at a time, up to
    128 in a group: the screened result equals the dense one, also when the
    points move away and back (chunks become zero and non-zero again)."""
    import paper_2512_16677_amd as q
    s = synth.water_like(walkers=2)
    rng = np.random.default_rng(shells)
    nuc = np.sort(np.r_[np.zeros(shells, int), rng.integers(1, 3, 40)])
    n = len(nuc)
    s.nucl_coord = np.array([[0.0, 0.0, 0.0], [9.0, 0.0, 0.0], [0.0, 14.0, 0.0]])
    s.shell_nucleus, s.shell_ang_mom = nuc, rng.integers(0, 2, n)
    s.shell_prim_offset = np.arange(n + 1)
    s.exponent, s.coefficient = 10.0 ** rng.uniform(-1.0, 2.5, n), np.ones(n)
    s.mo_coef = rng.normal(0.0, 0.1, size=(11, s.ao_num))
    ctx = q.Context.from_system(s, bits=24)
    for step in (0.0, 30.0, 3.0, 0.0):
        pts = (s.nucl_coord[rng.integers(0, 3, 200)] + rng.normal(size=(200, 3)) + step).reshape(1, 200, 3)
        ctx.set_point(pts)
        ctx.set_screening(False)
        dense = ctx.get_mo_vgl()
        ctx.set_screening(True)
        assert bool((ctx.get_mo_vgl() == dense).all())
    ctx.close()
