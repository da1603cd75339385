"""Device parameters that are refused leave the context's tables and copies of
C in place too: the call that can build none of them still runs, with the same
result, and so does a graph captured before (also when the refused C is larger)."""
import numpy as np
import pytest

import synth
from tests.test_gpu_ao_rows import system

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", ["C", "R"])
@pytest.mark.parametrize("mode", ["fp64", "mixed_f32", "mixed_bf16x3"])
@pytest.mark.parametrize("ao,times", [(25, 1), (25, 2), (25, 7), (1100, 7)])
def test_no_allocation_call_after_refused_parameters(bad, mode, ao, times):
    import paper_2512_16677_amd as q
    s = synth.water_like(walkers=4) if ao == 25 else system(ao)
    ctx = q.Context.from_system(s, mode=mode, points_on_device=True)
    before = ctx.get_mo_vgl()
    want, got = torch.empty_like(before), torch.empty_like(before)
    ctx.get_mo_vgl_noalloc(want)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ctx.get_mo_vgl_noalloc(got)
    C = torch.from_numpy(np.vstack([s.mo_coef] * times) + 1.0).cuda()
    R = torch.from_numpy(s.nucl_coord + 1.0).cuda()
    (C if bad == "C" else R).view(-1)[-1] = float("nan")
    with pytest.raises(q.QmkError) as e:
        ctx._set_params_device(R, C)
    assert e.value.status == q.QMK_NONFINITE
    assert "non-finite" in str(e.value)
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        got.zero_()
    ctx.get_mo_vgl_noalloc(got)
    assert torch.equal(got, want)
    assert torch.equal(ctx.get_mo_vgl(), before)
    ctx.close()
