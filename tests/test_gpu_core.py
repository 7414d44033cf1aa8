"""The small-state kernel at the edges of its straight-line forms: term slots
per lane of the secular solver (3, 6 or 9 for up to 24, 48 or 65 poles), tile
counts of its products, and the chunks in which it reads the passes' records.

Inputs: Gaussian snapshots, so every update has the full rank cap and all its
poles live.  Their singular values lie within a factor of ten of each other
and an update perturbs them by a few units of FP64 rounding of the largest,
so after at most 80 updates they agree with the oracle's to 1e-11 and one
predicted state to 1e-9, the bounds of the other FP64 comparisons.
"""
import numpy as np
import pytest

from oracle import odmd_oracle as O

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2311_18715_amd.odmd import ODMD


def run_against_the_oracle(n, r_max, updates, pairs, seed, shape=None):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((n, updates + 1))
    Y = rng.standard_normal((n, updates)) if pairs == "general" else X[:, 1:]
    g = ODMD(n, r_max, 1e-10, pairs=pairs, shape=shape)
    o = (O.OnlineDMDF1 if pairs == "general" else O.OnlineDMD)(n, r_max, 1e-10)
    Xd = torch.from_numpy(np.ascontiguousarray(X.T)).cuda()
    Yd = torch.from_numpy(np.ascontiguousarray(Y.T)).cuda()
    for j in range(updates):
        g.update(Xd[j], Yd[j])
        o.update(X[:, j], Y[:, j])
    s = g.state()
    assert s["r"] == o.r == min(r_max, updates)
    assert g.info().last_sweeps == 0        # the secular solver found every root
    np.testing.assert_allclose(s["sigma"], o.sigma, rtol=1e-11)
    ref = np.asarray(o.predict(1)).reshape(-1)
    got = g.predict(1).double().cpu().numpy().reshape(-1)
    assert np.linalg.norm(got - ref) <= 1e-9 * np.linalg.norm(ref)
    return g


@pytest.mark.parametrize("pairs", ["chained", "general"])
@pytest.mark.parametrize("r_max", [1, 7, 15, 16, 23, 24, 25, 47, 48, 49, 63, 64])
def test_every_rank_edge(r_max, pairs):
    run_against_the_oracle(900, r_max, r_max + 14, pairs, 100 + r_max)


@pytest.mark.parametrize("pairs", ["chained", "general"])
@pytest.mark.parametrize("blocks", [1, 13, 14, 130, 131, 261])
def test_record_chunks(blocks, pairs):
    """One record per 16 rows here: 13 slots of records, read ten at a time."""
    g = run_against_the_oracle(16 * blocks, 6, 24 if blocks > 1 else 12, pairs, 7 + blocks, (256, 16, 512))
    assert g.info().nblocks == blocks


@pytest.mark.parametrize("r_max", [15, 16, 33, 64])
@pytest.mark.parametrize("n", [700, 704, 8191, 8257, 16385])
def test_bf16_refold_gram_edges(n, r_max):
    """The Gram matrix of a rewritten BF16 basis with a ragged last tile, one,
    two and three workgroups of 8192 rows and 1 to 4 blocks of 16 columns.
    Rounded columns alone are off orthonormal by r 2^-9 / sqrt(n), at most
    5e-3 here; rows left out or counted twice would show as their share of
    the rows, at least 64 / 16385 per direction."""
    rng = np.random.default_rng(n + r_max)
    X = torch.from_numpy(rng.standard_normal((r_max + 40, n)).astype(np.float32)).cuda()
    g = ODMD(n, r_max, 1e-8, basis="bf16")
    stored = [0]
    for j in range(len(X) - 1):
        g.update(X[j], X[j + 1])
        stored.append(g.info().stored)
    assert any(b < a for a, b in zip(stored, stored[1:]))       # refolded
    U = g.basis_matrix().double()
    assert U.shape[1] == r_max
    orth = torch.linalg.norm(U.T @ U - torch.eye(r_max, dtype=U.dtype, device=U.device), 2).item()
    assert orth < (5e-3 if n < 8000 else 2e-3)


@pytest.mark.parametrize("pairs", ["chained", "general"])
@pytest.mark.parametrize("r_max", [1, 7, 15, 16, 23, 24, 25, 47, 48, 49, 63, 64])
def test_no_update_falls_back_to_jacobi(r_max, pairs):
    """The Jacobi fallback gives the same singular values, so a root that the
    secular solver missed shows only in the count of its sweeps: it is zero
    after every update, while the rank grows and at the cap."""
    rng = np.random.default_rng(300 + r_max)
    X = torch.from_numpy(rng.standard_normal((r_max + 15, 900))).cuda()
    Y = torch.from_numpy(rng.standard_normal((r_max + 15, 900))).cuda() if pairs == "general" else X[1:]
    g = ODMD(900, r_max, 1e-10, pairs=pairs)
    for j in range(r_max + 14):
        g.update(X[j], Y[j])
        assert g.info().last_sweeps == 0, j


@pytest.mark.parametrize("solver", ["secular", "jacobi"])
@pytest.mark.parametrize("pairs", ["chained", "general"])
@pytest.mark.parametrize("scale", [1e-140, 1e-100, 1e-60, 1e60, 1e100, 1e140])
@pytest.mark.parametrize("r_max", [7, 30, 64])
def test_snapshots_near_the_ends_of_the_exponent_range(r_max, scale, pairs, solver, monkeypatch):
    """Snapshots whose squares are in range and whose fourth powers are not:
    both solvers of the core work with squares of its entries times squares.
    The same bounds as at scale one, relative to the scale."""
    if solver == "jacobi":
        monkeypatch.setenv("ODMD_CORE_SVD", "jacobi")
    rng = np.random.default_rng(500 + r_max)
    updates = r_max + 14
    X = rng.standard_normal((900, updates + 1)) * scale
    Y = rng.standard_normal((900, updates)) * scale if pairs == "general" else X[:, 1:]
    g = ODMD(900, r_max, 1e-10, pairs=pairs)
    o = (O.OnlineDMDF1 if pairs == "general" else O.OnlineDMD)(900, r_max, 1e-10)
    Xd, Yd = (torch.from_numpy(np.ascontiguousarray(A.T)).cuda() for A in (X, Y))
    for j in range(updates):
        g.update(Xd[j], Yd[j])
        o.update(X[:, j], Y[:, j])
        assert (g.info().last_sweeps == 0) == (solver == "secular"), j
    g.sync()
    s = g.state()
    assert s["r"] == o.r == r_max
    np.testing.assert_allclose(s["sigma"], o.sigma, rtol=1e-11)
    U = g.basis_matrix()
    assert torch.linalg.norm(U.T @ U - torch.eye(r_max, dtype=U.dtype, device=U.device)).item() < 1e-12
    ref = np.asarray(o.predict(1)).reshape(-1) / scale
    got = g.predict(1).double().cpu().numpy().reshape(-1) / scale
    assert np.linalg.norm(got - ref) <= 1e-9 * np.linalg.norm(ref)


@pytest.mark.parametrize("pairs", ["chained", "general"])
@pytest.mark.parametrize("basis,power", [("f64", 400), ("f64", -400), ("f32", 110), ("bf16", 110)])
@pytest.mark.parametrize("solver", ["secular", "jacobi"])
def test_powers_of_two_scale_every_result_exactly(basis, power, pairs, solver, monkeypatch):
    """The core divided by a power of two and multiplied by it again gives the
    bits of the core at scale one; a BF16 basis takes the general SVD at its
    refolds.  (FP32's and BF16's residuals would leave their range downwards.)"""
    if solver == "jacobi":
        monkeypatch.setenv("ODMD_CORE_SVD", "jacobi")
    X = torch.from_numpy(np.random.default_rng(3).standard_normal((80, 700))).cuda().to(torch.float64 if basis == "f64" else torch.float32)
    a, b = (ODMD(700, 20, 1e-10, basis=basis, pairs=pairs) for _ in range(2))
    Z = X * 2.0 ** power
    for j in range(60):
        k = j + 1 if pairs == "chained" else (7 * j + 3) % 80
        a.update(X[j], X[k])
        b.update(Z[j], Z[k])
    a.sync(), b.sync()
    s, t = a.state(), b.state()
    assert s["r"] == t["r"] == 20 and a.info().last_sweeps == b.info().last_sweeps
    assert np.array_equal(s["sigma"], t["sigma"] * 2.0 ** -power)
    assert np.array_equal(s["atilde"], t["atilde"]) and np.array_equal(s["p_y"], t["p_y"] * 2.0 ** -power)
    assert torch.equal(a.basis_matrix(), b.basis_matrix())
    assert torch.equal(a.predict(6), b.predict(6) * 2.0 ** -power)
