"""Workloads of the online-DMD library as its users run them, for timing and for comparing outputs.

Each case is one way in which a program uses the public binding
(``paper_2311_18715_amd.odmd``): feeding snapshots to one large model,
forecasting after every snapshot, running the hybrid full-order/DMD loop,
analysing modes, rolling a model out, or advancing many streams at once and
serving their predictions.  Snapshots are planted linear streams (Gaussian
mode shapes times oscillating or decaying coefficients plus relative noise)
formed on the device from the seed.

``kind`` of a case:
  ingest    ``updates`` chained updates of one model, then the prediction of
            the next ``steps`` states; with 16 updates or more also the
            singular values, as a program that watches its rank reads them.
  general   the same on a general-pair model (trajectories that restart).
  hybrid    one step of the hybrid loop after a full-order step: update,
            rank, eigenvalues (convergence check), rollout of the horizon.
  modes     one update, then eigenvalues and eigenvectors.
  batch     ``updates`` batched updates of many streams, then the one-step
            prediction of each.
  serving   one round of a serving loop: a batched update of every stream,
            then the 100-state predictions that were asked for.

A chained model is fed from a ring of snapshots whose planted part has the
ring's length as its period, so that it can be fed for any number of passes;
its noise is more than its rank cap holds, as with measured or solver-limited
data, so that updates keep truncating and the basis keeps being rewritten.
"""
import math
import random

import numpy as np
import torch

from paper_2311_18715_amd.odmd import ODMD, handle_array, predict_batch, update_batch_ptrs

SNAP_BYTES = {"f64": 8, "f32": 4, "bf16": 4}       # snapshots and predictions
BASIS_BYTES = {"f64": 8, "f32": 4, "bf16": 2}      # stored basis
TOL = 1e-8
BF16_TOL = 2.0 ** -12                              # tolerance floor of a BF16 basis
RING = 96                                          # snapshots of one model's ring
BATCH_RING = 48                                    # snapshots of each stream's ring in a batch
SEGMENT = 24                                       # pairs of one trajectory before it restarts


def listed():
    return [
        # A small model (the planted n = 4096 stream) that forecasts one state after each snapshot: launches and latency.
        dict(name="forecast_f64_n4k", kind="ingest", n=4096, r=20, basis="f64", rank=7, noise=1e-6, updates=1, steps=1),
        # The benchmark stream's form: a 400 x 200 wake (u, v), FP64, rank cap 40; updates one at a time.
        dict(name="ingest_f64_n160k", kind="ingest", n=160000, r=40, basis="f64", rank=21, noise=1e-6, updates=64, steps=1),
        # The precision form's full size (3000 x 1000 wake) in each storage type: one large flow field.
        dict(name="ingest_f64_n6m", kind="ingest", n=6000000, r=64, basis="f64", rank=41, noise=1e-5, updates=16, steps=1),
        dict(name="ingest_f32_n6m", kind="ingest", n=6000000, r=64, basis="f32", rank=41, noise=1e-5, updates=16, steps=1),
        dict(name="ingest_bf16_n6m", kind="ingest", n=6000000, r=64, basis="bf16", rank=41, noise=1e-5, updates=16, steps=1),
        # Several trajectories of the wake-sized model (pairs that do not chain).
        dict(name="general_f64_n160k", kind="general", n=160000, r=40, basis="f64", rank=21, noise=1e-6, updates=32, steps=1),
        # One DMD step of the hybrid full-order/DMD loop at that size, horizon 16.
        dict(name="hybrid_f64_n160k", kind="hybrid", n=160000, r=40, basis="f64", rank=21, noise=1e-5, updates=1, steps=16),
        # Mode analysis of a model at the largest rank cap, an odd size (one row past whole tiles).
        dict(name="modes_f64_n20k", kind="modes", n=20033, r=64, basis="f64", rank=31, noise=1e-4, updates=1, steps=0),
        # The long rollout that ends a run, re-made after each new snapshot.
        dict(name="rollout500_f64_n160k", kind="ingest", n=160000, r=40, basis="f64", rank=21, noise=1e-6, updates=1, steps=500),
        # A 100-state forecast at the size of the paper's mesh, FP32 storage.
        dict(name="rollout100_f32_n586k", kind="ingest", n=585732, r=40, basis="f32", rank=21, noise=1e-5, updates=1, steps=100),
        # The many-stream form: 256 streams of 1e4 to 1e6 rows in batched steps.
        dict(name="batch256_f32", kind="batch", streams=256, n_lo=10000, n_hi=1000000, r_lo=16, r_hi=64, basis="f32", noise=1e-6,
             updates=16, steps=1, predicts=256),
        # A serving round: FP32 and BF16 streams of 1e4 to 2e6 rows, one request in ten a 100-state prediction.
        dict(name="serving_round_128", kind="serving", streams=128, n_lo=10000, n_hi=2000000, r_lo=16, r_hi=64, basis="mixed",
             noise=1e-6, updates=1, steps=100, predicts=13),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["ingest", "ingest", "ingest", "general", "hybrid", "modes", "rollout", "rollout", "batch", "serving"])
    if kind == "batch":
        return dict(kind="batch", streams=_log_int(rng, 8, 200), n_lo=10000, n_hi=_log_int(rng, 30000, 1000000), r_lo=16, r_hi=64,
                    basis=rng.choice(["f32", "f32", "f64"]), noise=1e-6, updates=rng.randint(4, 16), steps=1, predicts=rng.randint(1, 8))
    if kind == "serving":
        return dict(kind="serving", streams=_log_int(rng, 16, 128), n_lo=10000, n_hi=_log_int(rng, 100000, 2000000), r_lo=16, r_hi=64,
                    basis="mixed", noise=1e-6, updates=1, steps=rng.choice([20, 100, 100]), predicts=rng.randint(1, 13))
    basis = rng.choice(["f64", "f64", "f32", "f32", "bf16"])
    r = rng.randint(8, 64)
    c = dict(kind=kind, r=r, basis=basis, rank=2 * rng.randint(2, max(2, (r - 2) // 3)) + 1, noise=rng.choice([1e-6, 1e-5]))
    if kind == "ingest":
        n = _log_int(rng, 2000, 6000000)
        most = max(1, int(5e10 / (n * 80 * SNAP_BYTES[basis])))
        return dict(c, n=n, updates=rng.choice([1, min(most, rng.randint(8, 48))]), steps=rng.choice([1, 1, 4, 16]))
    if kind == "general":
        n = _log_int(rng, 2000, 1000000)
        return dict(c, n=n, basis=rng.choice(["f64", "f64", "f32"]), updates=rng.randint(1, 32), steps=rng.choice([1, 4, 16]))
    if kind == "rollout":
        n = _log_int(rng, 2000, 1000000)
        return dict(c, kind="ingest", n=n, updates=1, steps=_log_int(rng, 17, max(18, min(600, int(3e9 / (8 * n))))))
    n = _log_int(rng, 2000, 400000)
    return dict(c, kind=kind, n=n, basis="f64", noise=rng.choice([1e-5, 1e-4]), updates=1, steps=16 if kind == "hybrid" else 0)


# ---- inputs ---------------------------------------------------------------------------------------------------------


def _generator(seed, more=0):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + more * 7919 + 231118715) % (1 << 62))
    return g


def _io(basis):
    return torch.float64 if basis == "f64" else torch.float32


def _noisy(shapes, coeffs, noise, g, dtype):
    """coeffs @ shapes (snapshots as rows) plus noise relative to each snapshot, in the snapshot type."""
    out = torch.empty((coeffs.shape[0], shapes.shape[1]), dtype=dtype, device="cuda")
    for k0 in range(0, coeffs.shape[0], 16):
        X = torch.from_numpy(coeffs[k0:k0 + 16]).to("cuda", shapes.dtype) @ shapes
        if noise:
            scale = noise * torch.linalg.vector_norm(X, dim=1, keepdim=True) / math.sqrt(X.shape[1])
            X += scale * torch.randn(X.shape, generator=g, device="cuda", dtype=X.dtype)
        out[k0:k0 + 16] = X
    return out


def _ring(n, rank, noise, dtype, length, g, rng, amplitudes):
    """A ring of snapshots: a mean and (rank - 1) / 2 oscillations of whole frequencies of the ring; and its chained pairs."""
    pairs = rank // 2
    freq = rng.choice(np.arange(1, length // 2), size=pairs, replace=False) if amplitudes == "random" else np.arange(1, pairs + 1)
    amp = rng.uniform(0.3, 2.0, pairs) if amplitudes == "random" else 1.0 / (1.0 + np.arange(pairs)) ** 1.5
    phase = 2 * np.pi * np.outer(np.arange(length), freq) / length
    cols = [np.ones((length, 1))] if rank % 2 else []
    T = np.hstack(cols + [np.cos(phase) * amp, np.sin(phase) * amp])
    shapes = torch.randn((T.shape[1], n), generator=g, device="cuda", dtype=torch.float64 if amplitudes == "wake" else torch.float32)
    X = _noisy(shapes, T, noise, g, dtype)
    return X, [(k, (k + 1) % length) for k in range(length)]


def _trajectories(n, rank, noise, dtype, g, rng):
    """Trajectories of one decaying linear operator from fresh starts; the pairs inside each."""
    pairs, count = rank // 2, RING // SEGMENT
    lam = np.concatenate([(1.0 - 0.02 * (np.arange(pairs) + 1.0) / (pairs + 1)) * np.exp(2j * np.pi * 0.45 * (np.arange(pairs) + 1.0) / (pairs + 1)),
                          [0.999] * (rank % 2)])
    rows, pair, at = [], [], 0
    for _ in range(count):
        b = rng.standard_normal(len(lam)) + 1j * rng.standard_normal(len(lam))
        Z = b[None, :] * lam[None, :] ** np.arange(SEGMENT + 1)[:, None]
        rows.append(np.hstack([Z.real, -Z.imag]))
        pair += [(at + k, at + k + 1) for k in range(SEGMENT)]
        at += SEGMENT + 1
    shapes = torch.randn((2 * len(lam), n), generator=g, device="cuda", dtype=torch.float64)
    if rank % 2:
        shapes[-1] = 0.0                       # the real eigenvalue moves one real direction
    return _noisy(shapes, np.vstack(rows), noise, g, dtype), pair


def _single(case, seed):
    g, rng = _generator(seed), np.random.Generator(np.random.PCG64(int(seed)))
    if case["kind"] in ("general", "hybrid", "modes"):
        return _trajectories(case["n"], case["rank"], case["noise"], _io(case["basis"]), g, rng)
    return _ring(case["n"], case["rank"], case["noise"], _io(case["basis"]), RING, g, rng, "wake")


def _streams(case):
    """Sizes, rank caps, planted ranks and storage of the streams: part of the case, the same for every seed."""
    rng = random.Random("%(kind)s %(streams)d %(n_lo)d %(n_hi)d" % case)
    got = []
    for i in range(case["streams"]):
        n = _log_int(rng, case["n_lo"], case["n_hi"])
        basis = case["basis"] if case["basis"] != "mixed" else rng.choice(["f32", "bf16"])
        r = rng.choice([16, 32, 64]) if case["kind"] == "serving" else rng.randint(case["r_lo"], case["r_hi"])
        got.append((n, r, min(rng.randint(6, 30), r - 2), basis))
    return got


def _stream_ring(case, seed, i, n, rank, basis):
    rng = np.random.Generator(np.random.PCG64([int(seed), i]))
    return _ring(n, rank, case["noise"], _io(basis), BATCH_RING, _generator(seed, i + 1), rng, "random")[0]


def _warm(case):
    """Updates before the first pass: the rank has reached its cap and the basis has been rewritten."""
    return 40 if case["kind"] in ("batch", "serving") else case["r"] + 24


# ---- a user's program -----------------------------------------------------------------------------------------------


def prepare(case, seed):
    if case["kind"] in ("batch", "serving"):
        models, rings = [], []
        for i, (n, r, rank, basis) in enumerate(_streams(case)):
            rings.append(_stream_ring(case, seed, i, n, rank, basis))
            space = torch.empty(ODMD.state_bytes(n, r, basis), dtype=torch.uint8, device="cuda")
            models.append(ODMD(n, r, TOL, basis=basis, workspace=space))
        at = [np.array([x[k].data_ptr() for x in rings], dtype=np.uint64) for k in range(BATCH_RING)]
        asked = models[:case["predicts"]]
        flat = {d: torch.empty(sum(m.n * case["steps"] for m in asked if m.dtype == d), dtype=d, device="cuda") for d in {m.dtype for m in asked}}
        outs, used = [], {d: 0 for d in flat}
        for m in asked:                        # outputs in a space that the program keeps, as a server does
            size = m.n * case["steps"]
            outs.append(flat[m.dtype][used[m.dtype]:used[m.dtype] + size].view(case["steps"], m.n))
            used[m.dtype] += size
        state = dict(case=case, models=models, rings=rings, handles=handle_array(models), at=at, asked=asked, outs=outs, flat=flat, k=0)
        for _ in range(_warm(case)):
            _step_all(state)
        models[0].sync()
        return state
    X, pairs = _single(case, seed)
    kind = "general" if case["kind"] in ("general", "hybrid", "modes") else "chained"
    state = dict(case=case, X=list(X), pairs=pairs, model=ODMD(case["n"], case["r"], TOL, basis=case["basis"], pairs=kind), k=0)
    for _ in range(_warm(case)):
        _step(state)
    state["model"].sync()
    return state


def _step(state):
    a, b = state["pairs"][state["k"] % len(state["pairs"])]
    state["model"].update(state["X"][a], state["X"][b])
    state["k"] += 1


def _step_all(state):
    k = state["k"]
    update_batch_ptrs(state["handles"], state["at"][k % BATCH_RING], state["at"][(k + 1) % BATCH_RING])
    state["k"] = k + 1


def run(state):
    case = state["case"]
    if case["kind"] in ("batch", "serving"):
        for _ in range(case["updates"]):
            _step_all(state)
        predict_batch(state["asked"], [case["steps"]] * len(state["asked"]), state["outs"])
        return state["outs"] if len(state["outs"]) <= 64 else list(state["flat"].values())
    m = state["model"]
    for _ in range(case["updates"]):
        _step(state)
    if case["kind"] == "modes":
        lam, V = m.eigs(vectors=True)
        return {"lam": lam, "V": V}
    if case["kind"] == "hybrid":
        lam = m.eigs(vectors=False)[0] if m.info().r > 0 else None
        states = m.predict(case["steps"]) if m.info().r > 0 else None
        return {"lam": lam, "states": states}
    states = m.predict(case["steps"])
    if case["updates"] < 16:
        return {"states": states}
    return {"states": states, "sigma": m.state()["sigma"]}


# ---- what a pass cannot do without ----------------------------------------------------------------------------------


def work(case):
    """The basis read once and one column written per update (B beside U for general pairs), the pair read, the
    states written; two operations per basis entry for each of the three products of an update and each state."""
    if case["kind"] in ("batch", "serving"):
        models = _streams(case)
        # a BF16 basis keeps the planted directions, the others are filled to their cap by the noise
        rows = [(n, rank if b == "bf16" else r, BASIS_BYTES[b], SNAP_BYTES[b]) for n, r, rank, b in models]
        steps = [case["steps"] if i < case["predicts"] else 0 for i in range(len(rows))]
        ups, bases = case["updates"], 1
    else:
        rows = [(case["n"], case["r"], BASIS_BYTES[case["basis"]], SNAP_BYTES[case["basis"]])]
        steps, ups, bases = [case["steps"]], case["updates"], 1 if case["kind"] == "ingest" else 2
    total = flops = 0
    for (n, r, sb, sv), k in zip(rows, steps):
        total += ups * n * (bases * (r + 1) * sb + 2 * sv) + (n * (r * sb + k * sv) if k else 0)
        flops += ups * 6 * n * r * bases + 2 * n * r * k
        if case["kind"] in ("hybrid", "modes"):
            flops += 10 * r ** 3
    return {"bytes": total, "flops": flops}


# ---- the same in 64 bits --------------------------------------------------------------------------------------------


class _Reference:
    """Online DMD in textbook form and FP64: the column-append SVD update with an explicit basis (rows of U), Gram-Schmidt
    twice, numpy's SVD for the small problem, the shifted product of the right factor (chained pairs) or B = Y W."""

    def __init__(self, n, r_max, tol, general):
        self.r_max, self.tol, self.general = r_max, tol, general
        self.U = torch.zeros((0, n), dtype=torch.float64, device="cuda")
        self.B = torch.zeros((0, n), dtype=torch.float64, device="cuda") if general else None
        self.s, self.w, self.C = np.zeros(0), np.zeros(0), np.zeros((0, 0))

    def update(self, x, y):
        x, y = x.double(), y.double()
        U, r = self.U, len(self.s)
        p = U @ x
        e = x - p @ U
        p2 = U @ e
        e = e - p2 @ U
        rho = float(torch.linalg.vector_norm(e))
        keep = rho > self.tol * float(torch.linalg.vector_norm(x)) and rho > 0
        rho, q = (rho, e / rho) if keep else (0.0, torch.zeros_like(e))
        K = np.zeros((r + 1, r + 1))
        K[np.arange(r), np.arange(r)] = self.s
        K[:r, r], K[r, r] = (p + p2).cpu().numpy(), rho
        G, s, Vt = np.linalg.svd(K)
        k = min(self.r_max, int(np.count_nonzero(s > self.tol * s[0]))) if s[0] > 0 else 0
        G, V = G[:, :k], Vt.T[:, :k]
        self.U = torch.from_numpy(np.ascontiguousarray(G.T)).cuda() @ torch.cat([U, q[None]])
        if self.general:
            self.B = torch.from_numpy(np.ascontiguousarray(V.T)).cuda() @ torch.cat([self.B, y[None]])
        else:
            E = np.zeros((r + 1, r + 1))
            E[:r, :r], E[r, :r] = self.C, self.w
            self.C, self.w = V.T @ E @ V, V[r].copy()
        self.s, self.y = s[:k], y

    def operator(self):
        self.p = (self.U @ self.y).cpu().numpy()
        if self.general:
            return (self.U @ self.B.T).cpu().numpy() / self.s
        return (self.s[:, None] * self.C + np.outer(self.p, self.w)) / self.s

    def eigenvalues(self):
        lam = np.linalg.eigvals(self.operator()).astype(np.complex128)
        return lam[np.lexsort((-lam.imag, -np.abs(lam)))]

    def predict(self, steps):
        A, c, rows = self.operator(), self.p, []
        for _ in range(steps):
            c = A @ c
            rows.append(c)
        return torch.from_numpy(np.stack(rows)).cuda() @ self.U


def exact(case, seed):
    if case["kind"] in ("batch", "serving"):
        streams = _streams(case)[:case["predicts"]]
        if sum(n * case["steps"] for n, _, _, _ in streams) > 6e8 or len(streams) > 64:
            return None
        outs = []
        for i, (n, r, rank, basis) in enumerate(streams):
            X = _stream_ring(case, seed, i, n, rank, basis)
            m = _Reference(n, r, BF16_TOL if basis == "bf16" else TOL, False)
            for k in range(_warm(case) + case["updates"]):
                m.update(X[k % BATCH_RING], X[(k + 1) % BATCH_RING])
            outs.append(m.predict(case["steps"]))
        return outs
    X, pairs = _single(case, seed)
    m = _Reference(case["n"], case["r"], BF16_TOL if case["basis"] == "bf16" else TOL, case["kind"] != "ingest")
    for k in range(_warm(case) + case["updates"]):
        a, b = pairs[k % len(pairs)]
        m.update(X[a], X[b])
    if case["kind"] == "modes":
        return {"lam": m.eigenvalues(), "V": None}
    if case["kind"] == "hybrid":
        return {"lam": m.eigenvalues(), "states": m.predict(case["steps"])}
    if case["updates"] < 16:
        return {"states": m.predict(case["steps"])}
    return {"states": m.predict(case["steps"]), "sigma": m.s}
