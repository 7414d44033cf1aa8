"""Read-out kernels at the edges of their tiles, against the same product
formed from the model's own small state and basis.

The predicted states are U A~^k p_y.  The reference takes U from
odmd_get_basis (the wide FP64 read-out of the basis, another kernel than
the one under test for a few states), A~ and p_y from odmd_get_state, and
multiplies in FP64.  Tolerance: both sides sum at most 72 + k 64 FP64
products, so 1e-12 of the largest state entry covers their rounding, plus
one rounding of the output type; where the states come from the FP32 matrix
cores (five states and more on FP32 or BF16 storage), 73 FP32 roundings of
the sum of the products' magnitudes, bounded by sqrt(m) ||U row|| ||c||.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2311_18715_amd.odmd import ODMD, predict_batch


def model(n, r_max, basis, updates, seed=7):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    m = ODMD(n, r_max, 1e-8, basis=basis)
    X = torch.randn((updates + 1, n), generator=g, device="cuda", dtype=torch.float64).to(m.dtype)
    for k in range(updates):
        m.update(X[k], X[k + 1])
    m.sync()
    m._keep = X
    return m


def reference(m, steps):
    s = m.state()
    U = m.basis_matrix().cpu().numpy()
    c, rows, size = s["p_y"], [], []
    for _ in range(steps):
        c = s["atilde"] @ c
        rows.append(U @ c)
        size.append(np.linalg.norm(U, axis=1) * np.linalg.norm(c))
    return np.stack(rows), np.stack(size)


def check(m, got, steps):
    ref, size = reference(m, steps)
    got = got.double().cpu().numpy()
    tol = 1e-12 * np.abs(ref).max() + 0.0 * ref
    if m.dtype == torch.float32:
        tol = tol + 2.0 ** -24 * np.abs(ref)
        if steps > 4:
            tol = tol + 73 * 2.0 ** -24 * np.sqrt(72.0) * size
    assert got.shape == ref.shape and np.all(np.abs(got - ref) <= tol), np.max(np.abs(got - ref) / tol)


@pytest.mark.parametrize("basis", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("n", [1, 3, 63, 64, 65, 255, 257, 511, 513, 1025, 4099])
@pytest.mark.parametrize("steps", [1, 4, 5])
def test_few_states_at_tile_edges(basis, n, steps):
    m = model(n, min(n, 20), basis, 30)
    check(m, m.predict(steps), steps)


@pytest.mark.parametrize("basis", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("n", [37, 1024, 1031])
@pytest.mark.parametrize("steps", [16, 17, 32, 33, 64, 65, 96, 97, 128, 129, 200])
def test_state_blocks_and_stores(basis, n, steps):
    """Every number of state blocks per workgroup and a second block of them;
    n = 1024: states on whole lines (streaming stores), else ordinary ones;
    an output that starts one element off a line."""
    m = model(n, 20, basis, 30)
    check(m, m.predict(steps), steps)
    space = torch.empty(steps * n + 1, dtype=m.dtype, device="cuda")
    check(m, m.predict(steps, out=space[1:].view(steps, n)), steps)


@pytest.mark.parametrize("first", [1, 4, 5])
def test_a_few_states_of_many_streams_equal_each_streams_own(first):
    """Read-outs of up to 4 states share a launch per storage type and live
    bucket, longer ones do not: every stream's states equal its own call's
    bit for bit, whatever the mix, also two rows, one workgroup's rows and one
    more (256 threads of one FP64, two FP32 or four BF16 rows)."""
    specs = [(n, r, b) for b in ("f64", "f32", "bf16") for n, r in ((2, 1), (256, 6), (257, 6), (1025, 20), (3001, 40))]
    gen = torch.Generator(device="cuda").manual_seed(5)
    models = []
    for i, (n, r, b) in enumerate(specs):
        g = ODMD(n, r, 1e-10, basis=b)
        dt = torch.float64 if b == "f64" else torch.float32
        X = torch.randn((7 + 3 * i, n), generator=gen, device="cuda", dtype=dt)
        for k in range(len(X) - 1):
            g.update(X[k], X[k + 1])
        models.append(g)
    steps = [(first + i) % 7 + 1 for i in range(len(models))]
    one = [g.predict(k) for g, k in zip(models, steps)]
    many = predict_batch(models, steps)
    for a, b in zip(one, many):
        assert a.shape == b.shape and torch.equal(a.nan_to_num(7.0), b.nan_to_num(7.0))


@pytest.mark.parametrize("n,r", [(1, 1), (2, 2), (3, 3), (63, 4), (64, 4), (65, 3), (257, 2), (511, 4), (1025, 1), (4099, 4)])
@pytest.mark.parametrize("steps", [1, 4])
def test_few_states_equal_the_first_of_many(n, r, steps):
    """With a rank cap of at most four odmd_get_basis runs the few-state
    kernel too, so the reference here is the other one: the first states of a
    rollout of 17 (FP64 matrix cores: the same sums in another order)."""
    m = model(n, r, "f64", 12)
    got, ref = m.predict(steps), m.predict(17)[:steps]
    assert torch.isfinite(ref).all() and ref.abs().max() > 0
    assert (got - ref).abs().max() <= 1e-12 * ref.abs().max()


@pytest.mark.parametrize("basis", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("n", [1, 2, 3, 4])
@pytest.mark.parametrize("steps", [1, 4])
def test_few_states_of_a_few_rows(basis, n, steps):
    """Fewer rows than the matrix-core kernels' basis reference needs: with as
    many directions as rows nothing is truncated, and the states are A^k y
    with A = Y X^+ of all pairs.  A stored column is off by at most eps of
    itself and none is rewritten in 12 updates; that moves A by at most
    2 kappa sqrt(n) eps of it (kappa the condition of X), so k steps by twice k
    times that."""
    m = model(n, n, basis, 12)
    X = m._keep.double().cpu().numpy().T
    A = X[:, 1:] @ np.linalg.pinv(X[:, :-1])
    eps = {"f64": 1e-13, "f32": 2.0 ** -24, "bf16": 2.0 ** -9}[basis]
    got = m.predict(steps).double().cpu().numpy()
    state, kappa, size = X[:, -1], np.linalg.cond(X[:, :-1]), np.linalg.norm(A, 2)
    assert m.info().r == n and m.info().stored < m.info().capacity
    for k in range(1, steps + 1):
        state = A @ state
        assert np.linalg.norm(got[k - 1] - state) <= 4 * k * kappa * np.sqrt(n) * eps * size ** k * np.linalg.norm(X[:, -1])


def test_batched_few_states_are_finite():
    """Streams of a live rank have finite states, in a batch as by themselves
    (equal bits of two non-finite results would say nothing)."""
    models = [model(n, r, b, 12) for b in ("f64", "f32", "bf16") for n, r in ((2, 1), (256, 6), (1025, 9), (3001, 11))]
    assert all(m.info().r > 0 for m in models)
    for steps in (1, 4):
        for m, states in zip(models, predict_batch(models, [steps] * len(models))):
            assert torch.isfinite(states).all() and states.abs().max() > 0
            assert torch.equal(states, m.predict(steps))


@pytest.mark.parametrize("n", [600001, 1100032])
@pytest.mark.parametrize("steps", [2, 5, 10, 11, 16, 17])
def test_more_workgroups_for_few_states_of_many_rows(n, steps):
    """From 524,289 rows up to 10 FP64 states, and from 1,048,577 rows up to 16
    that start on whole lines (n = 1,100,032), take more workgroups per CU; the
    counts beyond take the usual ones.  Shares of unequal length either way."""
    m = model(n, 12, "f64", 16)
    check(m, m.predict(steps), steps)
