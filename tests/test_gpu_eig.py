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


def decoupled(r, c, scale, seed=23):
    """A model whose operator is diag(scale, c scale R), R random: one
    direction on rows of its own, with the largest singular value (index 0 of
    the reduced operator), and r - 1 others on the other rows.  Inner products
    between the two are exact zeros, so A~ decouples exactly."""
    n, q = 300, r - 1
    rng = np.random.default_rng(seed + r)
    X, Y = np.zeros((q + 9, n)), np.zeros((q + 9, n))
    X[0, :100] = 1e3 * rng.standard_normal(100)
    Y[0] = scale * X[0]
    A, C = rng.standard_normal((200, q)), rng.standard_normal((q, q + 8))
    B = rng.standard_normal((q, q)) / np.sqrt(q)
    X[1:, 100:] = (A @ C).T
    Y[1:, 100:] = (A @ (B @ C)).T * c * scale
    m = ODMD(n, r, 1e-10, pairs="general")
    for x, y in zip(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()):
        m.update(x, y)
    m.sync()
    return m


@pytest.mark.parametrize("r", [2, 3, 4, 6, 7, 21, 40, 64])
@pytest.mark.parametrize("c,scale", [(1.0, 1.0), (1e-56, 1.0), (1e-60, 1.0), (1e-67, 1.0), (1e-69, 1.0), (1e-80, 1.0), (1e-120, 1.0), (1e-135, 1.0),
                                     (1e-145, 1.0), (1e-180, 1e100), (1e-230, 1e120)])
def test_eigenvalues_of_a_block_far_below_the_rest(r, c, scale):
    """Every eigenvalue of a block that is far smaller than the matrix is
    found to the block's own precision (the bound of the dense test, for the
    block): squares and products of its entries lie below the smallest
    number where those of the matrix are of order one."""
    m = decoupled(r, c, scale)
    A = m.state()["atilde"]
    assert len(A) == r and np.all(A[0, 1:] == 0.0) and np.all(A[1:, 0] == 0.0)
    alone, _ = m.eigs(vectors=False)
    lam, V = m.eigs()
    assert np.array_equal(alone, lam) and np.all(np.isfinite(V))
    if c < 1.0:
        assert abs(lam[0] - A[0, 0]) <= 100 * r * EPS * abs(A[0, 0])
        lam, A = lam[1:], A[1:, 1:]
    lam, A = lam / (c * scale), A / (c * scale)
    ref, R = np.linalg.eig(A)
    bound = 100 * r * EPS * np.linalg.norm(A)
    for z, k in zip(ref, np.linalg.norm(np.linalg.inv(R), axis=1)):
        assert np.min(np.abs(lam - z)) <= 4 * k * bound


@pytest.mark.parametrize("r", [3, 4, 5, 8, 15, 16, 31, 63, 64])
def test_eigenvalues_of_a_cyclic_shift(r):
    """x_j = s_j e_j, y_j = s_j e_j+1: A~ is a cyclic permutation, which the
    trailing block's shifts leave as it is (only the exceptional shifts move
    it).  Its eigenvalues are the r-th roots of one, with condition one."""
    m = ODMD(300, r, 1e-10, pairs="general")
    E = torch.eye(r, 300, dtype=torch.float64, device="cuda") * torch.linspace(2.0, 1.0, r, dtype=torch.float64, device="cuda")[:, None]
    for j in range(r):
        m.update(E[j], torch.roll(E[j], 1) if j < r - 1 else torch.roll(E[j], 1 - r))
    m.sync()
    alone, _ = m.eigs(vectors=False)
    lam, V = m.eigs()
    A = m.state()["atilde"]
    bound = 100 * r * EPS * np.linalg.norm(A)
    assert np.array_equal(alone, lam)
    assert np.linalg.norm(A @ V - V * lam[None, :]) <= np.sqrt(r) * bound
    for z in np.exp(2j * np.pi * np.arange(r) / r):
        assert np.min(np.abs(lam - z)) <= bound
