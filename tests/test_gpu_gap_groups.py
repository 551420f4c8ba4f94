"""The gap's rows wait in the lanes of their group until all of them hold one: more rows to a group than it has lanes, a number that
does not divide, few rows, each kernel; against the sums formed from the device's own w and alphas in double."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("loss,kind,n,length,chunks", [
    ("hinge", "dense", 600011, 4, 3), ("logistic", "dense", 600011, 4, 3), ("squared", "dense", 70001, 20, 256), ("logistic", "dense", 77, 300, 2),
    ("logistic", "short", 5003, 3, 1), ("hinge", "short", 5003, 40, 1), ("squared", "short", 9001, 47, 2), ("logistic", "short", 12007, 60, 2),
    ("logistic", "mixed", 540007, 5, 256), ("hinge", "mixed", 61, 5, 4)])
def test_gap_is_the_sum_over_rows(loss, kind, n, length, chunks):
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    print("\ncase gap groups %s %s n=%d length=%d chunks=%d" % (loss, kind, n, length, chunks), flush=True)
    g = np.random.default_rng(n + length)
    y = (g.standard_normal(n) if loss == "squared" else np.where(g.random(n) < 0.5, -1, 1)).astype(np.float32)
    bounds = np.linspace(0, n, chunks + 1).astype(np.int64)
    if kind == "dense":
        d = length
        X = (g.standard_normal((n, d)) / np.sqrt(d)).astype(np.float32)
        p = Problem("gap", loss, n, d, 5.0 / n, y, bounds, X=X)
        dots = lambda w: X.astype(np.float64) @ w
    else:
        d = 1000
        lens = np.full(n, length)
        if kind == "mixed":                           # one row too long for the solver and the gap of short rows
            lens[n // 2] = 100
        start = g.integers(0, d - lens)
        rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
        col = (np.repeat(start, lens) + np.arange(rp[-1]) - np.repeat(rp[:-1], lens)).astype(np.int32)
        val = (g.standard_normal(rp[-1]) / np.sqrt(length)).astype(np.float32)
        p = Problem("gap", loss, n, d, 5.0 / n, y, bounds, row_ptr=rp, col=col, val=val)
        dots = lambda w: np.add.reduceat(val.astype(np.float64) * w[col], rp[:-1])
    r = binding.ChicleRound.from_problem(p, max_solvers=4)
    K = min(4, chunks)
    r.assign(K, (np.arange(chunks) % K).astype(np.int32))
    r.local_epoch(r.upload_perm([g.permutation(int(m)).astype(np.int32) for m in r.solver_rows()]))
    r.aggregate()
    P, D, _ = r.gap()
    w = r.get_w().astype(np.float64)
    a = np.concatenate([r.get_alpha(c) for c in range(chunks)]).astype(np.float64)
    z, lam = dots(w), 5.0 / n
    if loss == "hinge":
        primal, dual = np.maximum(0, 1 - y * z), a
    elif loss == "squared":
        primal, dual = 0.5 * (z - y) ** 2, a * y - 0.5 * a * a
    else:
        b = 1 - a
        primal = np.maximum(-y * z, 0) + np.log1p(np.exp(-np.abs(z)))
        dual = -(np.where(a > 0, a * np.log(np.maximum(a, 1e-300)), 0) + np.where(b > 0, b * np.log(np.maximum(b, 1e-300)), 0))
    ref = 0.5 * lam * (w @ w) + primal.mean(), -0.5 * lam * (w @ w) + dual.mean()
    print("primal %.3e dual %.3e" % (abs(P - ref[0]) / abs(ref[0]), abs(D - ref[1]) / max(abs(ref[1]), abs(ref[0]))), flush=True)
    # w is read out as floats, 2^-24 off each, where the device has it in double; a row's dot product carries sqrt(length) of them
    tol = 2.0 ** -24 * 4 * np.sqrt(length) * max(1.0, float(np.abs(w).max()))
    assert abs(P - ref[0]) <= tol * (abs(ref[0]) + 1) and abs(D - ref[1]) <= tol * (abs(ref[0]) + 1)
    r.close()
