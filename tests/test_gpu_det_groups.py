"""Determinants and adjugates of 5 <= n <= 32, several matrices per wavefront:
batches that end inside a wavefront or a workgroup, and matrices that take the
general path (singular, or with a NaN) beside ordinary ones of the same
wavefront.  Tolerances as for one matrix at a time: 1e-11 relative for these
well-conditioned inputs, 1e-10 of the largest cofactor for the singular ones."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 8, 9, 15, 16, 17, 31, 32])
@pytest.mark.parametrize("extra", [-1, 0, 1])
def test_ragged_batches_and_mixed_wavefronts(n, extra):
    import paper_2512_16677_amd as q
    group = 8 if n <= 8 else (4 if n <= 16 else 2)  # matrices per wavefront
    batch = 4 * group + group + extra               # a workgroup and about one wavefront
    rng = np.random.default_rng(1000 * n + extra + 1)
    a = rng.normal(size=(batch, n, n)) + 2.0 * np.sqrt(n) * np.eye(n)
    a = a[:, rng.permutation(n)]                     # pivots off the diagonal
    singular = [1, batch - 1]
    a[1, :, 2] = 0.0
    a[batch - 1, 3] = a[batch - 1, 0]
    a[group, 1, n - 1] = np.nan
    c = q.Context()
    det, adj = c.det_adj(torch.from_numpy(a).cuda())
    c.close()
    det, adj = det.cpu().numpy(), adj.cpu().numpy()
    assert np.isnan(det[group])
    rest = [b for b in range(batch) if b != group]
    rdet, radj = oracle.det_adj(a[rest])
    assert np.all(np.isfinite(adj[rest]))
    for k, b in enumerate(rest):
        if b in singular:
            assert det[b] == 0.0
            assert np.abs(adj[b] - radj[k]).max() <= 1e-10 * np.abs(radj[k]).max(), b
        else:
            assert abs(det[b] - rdet[k]) <= 1e-11 * abs(rdet[k]), b
            assert np.abs(adj[b] - radj[k]).max() <= 1e-11 * np.abs(radj[k]).max(), b
