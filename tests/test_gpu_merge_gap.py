"""The merge in slices of solvers, whose last slice writes the float mirror, and the gap, whose last workgroup adds everything
up: columns at the edges of a workgroup's, one solver and many, several rounds on the same counters, after a call without the
sums as well."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n,m,K", [(1, 70, 1, 1), (31, 90, 3, 2), (2048, 400, 12, 3), (2049, 700, 60, 5), (70001, 3000, 20, 40), (300000, 300, 40, 30),
                                     (2000000, 1200, 40, 24), (40, 900, 0, 4)])
def test_merge_and_gap(d, n, m, K):
    import torch
    import paper_1909_04885_amd as chicle
    assert torch.cuda.is_available()
    print("\ncase merge and gap d=%d n=%d m=%d K=%d" % (d, n, m, K), flush=True)
    g = np.random.default_rng(11)
    dense = m == 0
    lam, l1 = 1.0 / n, 0.01 if d < 100000 else 1e-4      # (a step moves a column by about 1e-3 in the larger ones)
    y = g.standard_normal(n).astype(np.float32)
    X = np.zeros((n, d), dtype=np.float32) if dense else None
    bounds = np.linspace(0, n, K + 1).astype(np.int64)
    r = chicle.ChicleRound("squared", n, d, lam, K, K, dense, n * (d if dense else m))
    if dense:
        X[:] = g.standard_normal((n, d))
    else:
        col = np.concatenate([np.sort(g.choice(d, m, replace=False)) for _ in range(n)]).astype(np.int32)
        val = g.standard_normal(n * m).astype(np.float32)
        rp = m * np.arange(n + 1, dtype=np.int64)
    for k in range(K):
        a, b = bounds[k], bounds[k + 1]
        if dense:
            r.load_chunk_dense(k, X[a:b], y[a:b])
        else:
            r.load_chunk_csr(k, rp[a:b + 1] - rp[a], col[rp[a]:rp[b]], val[rp[a]:rp[b]], y[a:b])
    r.set_l1(l1)
    r.assign(K, np.arange(K, dtype=np.int32))
    v = np.zeros(d)                                     # the dual image, in double
    eps = 2.0 ** -24
    for rnd in range(3):
        r.local_epoch(r.upload_perm([g.permutation(int(x)) for x in r.solver_rows()]))
        parts = [r.get_delta_w(k).astype(np.float64) for k in range(K)]
        v += np.sum(parts, axis=0)
        r.aggregate()
        w = np.sign(v) * np.maximum(np.abs(v) - l1, 0.0)
        # float sums of up to K terms, scaled, three rounds of them; the mirror's own rounding
        slack = (rnd + 1) * (K + 2) * eps * (np.abs(parts).sum(axis=0).max() + np.abs(v).max())
        got = r.get_w().astype(np.float64)
        assert np.all(np.abs(got - w) <= slack + eps * np.abs(w))
        if rnd == 1:
            continue                                    # the next pass runs the rows' part alone
        for _ in range(2):
            P, D, gap = r.gap()
            # from the device's own state: sums in double, of a w that the mirror holds to 2^-24 of each column
            z = X.astype(np.float64) @ got if dense else (val.astype(np.float64) * got[col]).reshape(n, m).sum(axis=1)
            dz = eps * (np.abs(X).astype(np.float64) @ np.abs(got) if dense else np.abs(val.astype(np.float64) * got[col]).reshape(n, m).sum(axis=1))
            alpha = np.concatenate([r.get_alpha(k) for k in range(K)]).astype(np.float64)
            norm = lam * (0.5 * got @ got + l1 * np.abs(got).sum())
            P_ref = 0.5 * np.mean((z - y) ** 2) + norm
            D_ref = -np.mean(0.5 * alpha ** 2 - alpha * y) - 0.5 * lam * (got @ got)
            off = 2.5 * eps * norm + (n + d) * 2.0 ** -52 * (abs(P_ref) + np.mean(0.5 * alpha ** 2 + np.abs(alpha * y)))
            off_P = off + np.mean(np.abs(z - y) * dz + 0.5 * dz ** 2)
            print("P %.1e of %.1e, D %.1e of %.1e, norms %.1e" % (abs(P - P_ref), off_P, abs(D - D_ref), off, norm), flush=True)
            assert abs(P - P_ref) <= off_P and abs(D - D_ref) <= off and gap == P - D
            assert min(lam * 0.5 * got @ got, norm) > 100 * off_P          # (norms left out would show)
    r.close()


@pytest.mark.parametrize("dense", [True, False])
def test_gap_of_65535_chunks(dense):
    """As many chunks of a row as a grid's second dimension has places: the norms have workgroups beside the chunks'."""
    import torch
    import paper_1909_04885_amd as chicle
    assert torch.cuda.is_available()
    print("\ncase gap of 65535 chunks, %s" % ("dense" if dense else "sparse"), flush=True)
    g = np.random.default_rng(5)
    n, d, m, K = 65535, 40, 8, 86
    lam = 0.05
    y, alpha = g.standard_normal(n).astype(np.float32), g.standard_normal(n).astype(np.float32)
    col = np.sort(np.argsort(g.random((n, d)), axis=1)[:, :m], axis=1).astype(np.int32)
    X = g.standard_normal((n, d)).astype(np.float32)
    if not dense:
        keep = np.zeros((n, d), dtype=bool)
        np.put_along_axis(keep, col, True, axis=1)
        X[~keep] = 0.0
    r = chicle.ChicleRound("squared", n, d, lam, n, K, dense, n * (d if dense else m))
    rp = np.array([0, m], dtype=np.int32)
    for i in range(n):
        if dense:
            r.load_chunk_dense(i, X[i:i + 1], y[i:i + 1], alpha[i:i + 1])
        else:
            r.load_chunk_csr(i, rp, col[i], X[i, col[i]], y[i:i + 1], alpha[i:i + 1])
    r.assign(K, (np.arange(n) % K).astype(np.int32))
    w = g.standard_normal(d).astype(np.float32)
    r.set_w(w)
    w, z, a = w.astype(np.float64), X.astype(np.float64) @ w.astype(np.float64), alpha.astype(np.float64)
    P_ref = 0.5 * np.mean((z - y) ** 2) + 0.5 * lam * (w @ w)
    D_ref = -np.mean(0.5 * a ** 2 - a * y) - 0.5 * lam * (w @ w)
    for _ in range(2):
        P, D, gap = r.gap()
        # doubles added in another order: n + d terms of one sign (the dual's: of at most 8 times its value)
        tol = (n + d) * 2.0 ** -52
        print("P %.3e D %.3e" % (abs(P / P_ref - 1), abs(D / D_ref - 1)), flush=True)
        assert abs(P - P_ref) <= tol * P_ref and abs(D - D_ref) <= 8 * tol * abs(D_ref) and gap == P - D
    r.close()


def test_merge_adds_in_double():
    """Sixteen solvers in slices of several, thickly occupied vectors: what reaches the shared vector is the sum of the updates in
    double, however many of them a slice adds up."""
    import torch
    import paper_1909_04885_amd as chicle
    assert torch.cuda.is_available()
    print("\ncase merge in double", flush=True)
    g = np.random.default_rng(23)
    n, d, m, K = 32000, 300000, 48, 16           # (sixteen: a solver's update is its vector over K, without a rounding)
    col = (np.arange(m) * (d // m) + g.integers(0, d // m, (n, m))).astype(np.int32)
    val = g.standard_normal((n, m)).astype(np.float32)
    y = np.where(g.random(n) < 0.5, -1.0, 1.0).astype(np.float32)
    r = chicle.ChicleRound("hinge", n, d, 1.0 / n, K, K, False, n * m)
    rows = n // K
    for k in range(K):
        a, b = k * rows, (k + 1) * rows
        r.load_chunk_csr(k, m * np.arange(rows + 1), col[a:b].reshape(-1), val[a:b].reshape(-1), y[a:b])
    r.assign(K, np.arange(K, dtype=np.int32))
    total, size = np.zeros(d), np.zeros(d)
    for _ in range(2):
        r.local_epoch(r.upload_perm([g.permutation(rows) for _ in range(K)]))
        for k in range(K):
            part = r.get_delta_w(k).astype(np.float64)
            total += part
            size += np.abs(part)
        r.aggregate()
        # the mirror's rounding to float, and roundings of doubles
        off = np.abs(r.get_w().astype(np.float64) - total)
        print("beyond the bound: %d of %d columns" % (np.count_nonzero(off > 2.0 ** -24 * np.abs(total) + 2.0 ** -47 * size), d), flush=True)
        assert np.all(off <= 2.0 ** -24 * np.abs(total) + 2.0 ** -47 * size)
    r.close()
