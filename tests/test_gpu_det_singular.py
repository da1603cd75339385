"""Determinants and adjugates of 5 <= n <= 32 outside the well-conditioned
matrices: singular ones at every place of a wavefront (a whole batch, the last
one alone, beside ordinary ones), badly scaled and nearly singular ones, pivots at
the ends of the range and NaNs.  Singular matrices: det = 0 and the adjugate
within 1e-10 of its largest entry (0 for rank n - 2), as for one at a time; the
others against exact rational arithmetic, within 64 n cond(A) eps of the largest
entry, cond in the infinity norm after rows and columns are scaled to a largest
entry of 1 (elimination does not notice scalings by powers of two).  With a
pivot below the normal numbers the entries that contain it are products of such
numbers, which hold few bits: they are finite."""
from fractions import Fraction

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def det_adj(a):
    import paper_2512_16677_amd as q
    c = q.Context()
    det, adj = c.det_adj(torch.from_numpy(np.ascontiguousarray(a)).cuda())
    c.close()
    return det.cpu().numpy(), adj.cpu().numpy()


@pytest.mark.parametrize("n", [5, 7, 8, 9, 16, 17, 31, 32])
@pytest.mark.parametrize("batch", [1, 3, 37])
def test_all_singular(n, batch):
    rng = np.random.default_rng(n * 100 + batch)
    kinds = {}
    a = rng.normal(size=(batch, n, n))
    kinds["zero row"] = a.copy()
    kinds["zero row"][:, rng.integers(n)] = 0.0
    kinds["zero column"] = a.copy()
    kinds["zero column"][:, :, rng.integers(n)] = 0.0
    kinds["last column zero"] = a.copy()
    kinds["last column zero"][:, :, n - 1] = 0.0
    kinds["first column zero"] = a.copy()
    kinds["first column zero"][:, :, 0] = 0.0
    kinds["equal rows"] = a.copy()
    kinds["equal rows"][:, 3] = kinds["equal rows"][:, 1]
    shift = np.eye(n, k=1)  # rank n - 1; its only cofactor is the lower left corner
    kinds["shift"] = np.broadcast_to(shift, a.shape).copy()
    for name, m in kinds.items():
        det, adj = det_adj(m)
        assert np.all(det == 0.0), name
        if name == "shift":
            ref = np.zeros((batch, n, n))
            ref[:, 0, n - 1] = (-1.0) ** (n - 1)
        else:
            ref = oracle.det_adj(m)[1]
        top = np.abs(ref).max(axis=(1, 2), keepdims=True)
        assert np.all(np.abs(adj - ref) <= 1e-10 * top), name
    two = a.copy()
    two[:, 0] = two[:, n - 1] = 0.0
    for m in (np.zeros_like(a), two):
        det, adj = det_adj(m)
        assert np.all(det == 0.0) and np.all(adj == 0.0)


def exact(a):
    """(det, adj) of one matrix in rational arithmetic, as floats (python's own
    conversion is correctly rounded)."""
    n = len(a)
    m = [[Fraction(float(x)) for x in r] + [Fraction(int(i == j)) for j in range(n)] for i, r in enumerate(a)]
    d = Fraction(1)
    for k in range(n):
        p = next(i for i in range(k, n) if m[i][k])
        if p != k:
            m[k], m[p], d = m[p], m[k], -d
        d *= m[k][k]
        m[k] = [x / m[k][k] for x in m[k]]
        for i in range(n):
            if i != k and m[i][k]:
                f = m[i][k]
                m[i] = [x - f * y for x, y in zip(m[i], m[k])]
    return float(d), np.array([[float(d * m[i][n + j]) for j in range(n)] for i in range(n)])


@pytest.mark.parametrize("n", [5, 8, 9])
@pytest.mark.parametrize("kind", ["rows", "columns", "both", "near", "large pivot", "small pivot"])
def test_scaled_and_nearly_singular(n, kind):
    rng = np.random.default_rng(n)
    a = rng.integers(-2 ** 20, 2 ** 20, size=(6, n, n)) / 2.0 ** 20
    r = 2.0 ** rng.integers(-20, 20, size=(6, n, 1))
    c = 2.0 ** rng.integers(-20, 20, size=(6, 1, n))
    if kind == "near":
        a[:, 2] = a[:, 0] + a[:, 1] + 2.0 ** -30 * a[:, 2]
    b = a * (r if kind in ("rows", "both") else 1.0) * (c if kind in ("columns", "both") else 1.0)
    if kind in ("large pivot", "small pivot"):  # one pivot whose reciprocal is not a normal number
        s = 2.0 ** 1023 if kind == "large pivot" else 2.0 ** -1040
        b = a * 2.0 ** -8
        b[:, 0, :] = b[:, :, 0] = 0.0
        b[:, 0, 0] = 1.5 * s
    det, adj = det_adj(b)
    for k in range(len(b)):
        rd, ra = exact(b[k])
        scaled = b[k] / np.abs(b[k]).max(axis=1, keepdims=True)
        scaled = scaled / np.abs(scaled).max(axis=0, keepdims=True)
        tol = 64 * n * np.linalg.cond(scaled, np.inf) * 2.0 ** -53
        assert np.isfinite(det[k]) and np.all(np.isfinite(adj[k])), k
        if kind == "small pivot":
            assert abs(adj[k, 0, 0] - ra[0, 0]) <= tol * abs(ra[0, 0]), k
            continue
        assert abs(det[k] - rd) <= tol * abs(rd), k
        if kind == "large pivot":  # the two diagonal blocks are of their own sizes
            assert abs(adj[k, 0, 0] - ra[0, 0]) <= tol * abs(ra[0, 0]), k
            ra, got = ra[1:, 1:], adj[k, 1:, 1:]
        else:
            got = adj[k]
        assert np.abs(got - ra).max() <= tol * np.abs(ra).max(), k


@pytest.mark.parametrize("n", [5, 8, 16, 17, 32])
def test_nan_in_a_column_of_zeros(n):
    rng = np.random.default_rng(n)
    a = rng.normal(size=(9, n, n))
    a[:, :, 1] = 0.0
    a[:, n - 1, 1] = np.nan
    det, _ = det_adj(a)
    assert np.all(np.isnan(det))
