"""odmd_eigs over the ranks at which its bulge count, parts and tiles change.

Inputs: random pairs of a random r x r operator seen through n = 300 rows
(general pairs), so that A~ is a dense random matrix of that rank.  The
reduced operator is read back and the eigenpairs are checked against it:
the QR iteration is backward stable, so ||A~ V - V Lambda||_F is at most a
modest multiple of r eps ||A~||_F (100 taken, times sqrt(r) for the r unit
columns), the columns of V have norm one to r eps, and each eigenvalue that
numpy finds has one within the same residual times its condition number.
Scaled streams put A~ near the ends of the exponent range.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2311_18715_amd.odmd import ODMD

EPS = 2.0 ** -52


def model(r, scale, seed=11):
    n, count = 300, r + 8
    rng = np.random.default_rng(seed + r)
    A = rng.standard_normal((n, r))
    C = rng.standard_normal((r, count))
    B = rng.standard_normal((r, r)) / np.sqrt(r)
    X = torch.from_numpy(np.ascontiguousarray((A @ C).T)).cuda()
    Y = torch.from_numpy(np.ascontiguousarray((A @ (B @ C)).T)).cuda() * scale
    m = ODMD(n, r, 1e-10, pairs="general")
    for x, y in zip(X, Y):
        m.update(x, y)
    m.sync()
    return m


@pytest.mark.parametrize("scale", [1.0, 1e-120, 1e120])
@pytest.mark.parametrize("r", [1, 2, 3, 4, 5, 9, 10, 15, 19, 20, 33, 63, 64])
def test_eigenpairs_of_the_reduced_operator(r, scale):
    m = model(r, scale)
    alone, none = m.eigs(vectors=False)
    A = m.state()["atilde"] / scale
    lam, V = m.eigs()
    assert none is None and np.array_equal(alone, lam) and len(lam) == len(A) == r
    lam = lam / scale
    bound = 100 * r * EPS * np.linalg.norm(A)
    assert np.linalg.norm(A @ V - V * lam[None, :]) <= np.sqrt(r) * bound
    assert np.max(np.abs(np.linalg.norm(V, axis=0) - 1.0)) <= 10 * r * EPS
    top = V[np.argmax(np.abs(V), axis=0), np.arange(r)]
    assert np.all(top.imag == 0.0) and np.all(top.real > 0.0)
    ref, R = np.linalg.eig(A)
    cond = np.linalg.norm(np.linalg.inv(R), axis=1)      # 1 / |y.x| of unit eigenvectors
    for z, k in zip(ref, cond):
        assert np.min(np.abs(lam - z)) <= 4 * k * bound
    key = [(-abs(z), -z.imag) for z in lam * scale]
    assert all(a[0] <= b[0] for a, b in zip(key, key[1:]))
