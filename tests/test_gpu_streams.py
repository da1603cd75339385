"""Calls that are still waiting on a side stream keep the inputs that they were
made with: nuclei (which change the order of the AO rows from 1024 AOs on), MO
coefficients, precision, points, occupations and Jastrow coefficients are set
anew behind a queue of other work, and every result equals, bit for bit, the one
of the same calls with a wait after each.  With two streams the change comes
between a call on one and a call on the other."""
import numpy as np
import pytest

import synth
from tests.test_gpu_ao_rows import system

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def changes(q, ctx, s):
    xyz = np.ascontiguousarray(s.nucl_coord[:, [1, 0, 2]])
    coef = np.ascontiguousarray(s.mo_coef[:, ::-1])
    dev = [torch.from_numpy(a.copy()).cuda() for a in (xyz, coef)]
    return {"nuclei": lambda: ctx.set_nucleus(xyz), "coefficients": lambda: ctx.set_mo_coef(coef),
            "precision": lambda: ctx.set_precision(24, "mixed_f32"),
            "device parameters": lambda: ctx._set_params_device(*dev),
            "points": lambda: ctx.set_point(s.elec_coord + 0.5), "others": lambda: None}


def calls(ctx, s, w, second):
    occ = np.linspace(0.5, 2.0, s.mo_num)[::-1 if second else 1].copy()
    out = [ctx.get_mo_vgl(), ctx.get_mo_value(), ctx.get_density(occ), *ctx.adjoint(w).values()]
    import paper_2512_16677_amd as q
    c = np.linspace(-1.0, 1.0, q.jastrow_een_terms(4) * s.nucl_num).reshape(-1, s.nucl_num)
    return out + [ctx.jastrow_een(4, 0.8, -c if second else c)]


def run(q, s, w, screening, what, first, then, load):
    ctx = q.Context.from_system(s)
    ctx.set_screening(screening)
    change = changes(q, ctx, s)[what]
    with torch.cuda.stream(first):
        calls(ctx, s, w, False)  # tables, tiles, workspaces
    torch.cuda.synchronize()
    with torch.cuda.stream(first):
        if load is not None:
            for _ in range(12):
                load = load @ load
        a = calls(ctx, s, w, False)
    if load is None:
        torch.cuda.synchronize()
    with torch.cuda.stream(then):
        change()
        b = calls(ctx, s, w, True)
    torch.cuda.synchronize()
    got = [x.cpu() for x in a + b]
    ctx.close()
    return got


# a change of points or occupations alone leaves the order of the calls on two
# streams, which share the context's arrays, to the caller
ONE = ["nuclei", "coefficients", "precision", "device parameters", "points", "others"]
CASES = [(1, what) for what in ONE] + [(2, what) for what in ONE[:4]]


@pytest.mark.parametrize("streams,what", CASES)
@pytest.mark.parametrize("ao,screening", [(60, False), (1100, False), (1100, True)])
def test_enqueued_calls_keep_their_inputs(streams, what, ao, screening):
    import paper_2512_16677_amd as q
    s = system(ao, seed=ao)
    w = torch.from_numpy(synth.adjoint_weights(s, seed=8)).cuda()
    load = torch.eye(4096, device="cuda")
    side = torch.cuda.Stream()
    then = torch.cuda.Stream() if streams == 2 else side
    torch.cuda.synchronize()
    waited = run(q, s, w, screening, what, side, side, None)
    queued = run(q, s, w, screening, what, side, then, load)
    for k, (x, y) in enumerate(zip(waited, queued)):
        assert torch.equal(x, y), k
