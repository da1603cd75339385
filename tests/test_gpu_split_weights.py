"""BF16x3 weights at every alignment of a weight: rows of N weights around the
eight that one thread splits, from a buffer that starts on a 16-byte boundary
or one weight after it.  The gradients are the same bit for bit, alone and in a
batch, and within the mode's bound of the oracle."""
import numpy as np
import pytest

import oracle
import synth
from tests.helpers import grad_err
from tests.test_gpu_mixed import TOL

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("mo", [1, 7, 8, 9, 15, 25])
def test_weights_at_any_alignment(mo, dtype):
    import paper_2512_16677_amd as q
    s = synth.water_like(walkers=3)
    s.mo_coef = np.random.default_rng(mo).normal(0.0, 0.2, size=(mo, s.ao_num))
    w = torch.from_numpy(synth.adjoint_weights(s, seed=4)).to(dtype).cuda()
    shifted = torch.empty(w.numel() + 1, dtype=dtype, device="cuda")[1:].view_as(w)
    shifted.copy_(w)
    got = []
    for wi in (w, shifted):
        ctx = q.Context.from_system(s, mode="mixed_bf16x3", bits=24)
        ctx.get_mo_vgl()
        g = ctx.adjoint(wi)
        b = q.Batch([ctx, ctx])
        _, gb = b.run(dtype=dtype, ws=[wi, w])
        torch.cuda.synchronize()
        got.append([g[k].clone() for k in sorted(g)] + [x[k].clone() for x in gb for k in sorted(x)])
        b.close()
        ctx.close()
    for a, b in zip(*got):
        assert torch.equal(a, b)
    r = oracle.adjoint(s, w.double().cpu().numpy(), B=24)
    for v, k in zip(got[0], sorted(("d_coef", "d_elec", "d_nucl"))):
        assert grad_err(v.cpu().numpy().reshape(r[k].shape), r[k], r[k + "_abs"]) <= TOL["mixed_bf16x3"]["grad"]
