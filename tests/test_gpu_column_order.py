"""Long rows: the copy of the entries by column that the gap's row pass and the merge stream over.  Rows on both sides of a block of
16384, columns in several segments of 262144, a last bucket that is not full, one bucket that holds everything (merged through the
private vectors), solvers by name in turn, updates read out between pass and merge; and the same with shorter rows, whose dot products
are formed row by row."""
import numpy as np
import pytest

from harness import TOL_DW, dw_floor, gap_tolerance, rel_l2

pytestmark = pytest.mark.gpu


# (dots, merge: whether these go over the entries by column)
@pytest.mark.parametrize("loss,n,d,length,popular,l1,by_name,dots,merge", [
    ("hinge", 16400, 600011, 100, 0, 0.0, False, False, True), ("squared", 321, 5003, 130, 0, 0.0, True, False, True),
    ("logistic", 500, 300001, 200, 0, 0.0, False, False, True), ("hinge", 700, 300001, 150, 900, 0.0, True, False, False),
    ("squared", 40, 20000003, 300, 0, 0.0, False, True, False), ("hinge", 321, 262145, 130, 0, 0.02, True, False, True),
    ("squared", 2500, 40009, 400, 0, 0.0, False, False, False),
    ("hinge", 16400, 600011, 300, 0, 0.0, False, True, None), ("squared", 500, 5003, 1200, 0, 0.0, True, True, None),
    ("logistic", 500, 300001, 900, 0, 0.0, False, True, True), ("hinge", 700, 300001, 900, 1000, 0.0, True, True, None),
    ("squared", 40, 20000003, 3000, 0, 0.0, False, True, False), ("hinge", 321, 262145, 1000, 0, 0.02, True, True, True),
    ("squared", 2500, 40009, 900, 0, 0.0, False, True, None)])
def test_passes_by_column(oracle_mod, loss, n, d, length, popular, l1, by_name, dots, merge):
    import torch
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    assert torch.cuda.is_available()
    print("\ncase columns %s n=%d d=%d length=%d popular=%d" % (loss, n, d, length, popular), flush=True)
    g = np.random.default_rng(n + d)
    lens = g.integers(length // 2, length + length // 2 + 8, n)
    rows = [np.sort(g.choice(popular or d, min(m, popular or d), replace=False)) if popular or d < 10 ** 5
            else np.unique(g.integers(0, d, m)) for m in lens]
    lens, col = [len(c) for c in rows], np.concatenate(rows).astype(np.int32)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    val = (g.standard_normal(len(col)) / np.sqrt(length)).astype(np.float32)
    y = (g.standard_normal(n) if loss == "squared" else np.where(g.random(n) < 0.5, -1, 1)).astype(np.float32)
    bounds = np.unique(np.concatenate([np.arange(0, n, max(7, n // 9)), [n]])).astype(np.int64)
    p = Problem("columns", loss, n, d, 20.0 / n, y, bounds, row_ptr=rp, col=col, val=val)
    assert len(col) > 96 * n
    K = min(5, len(bounds) - 1)
    r = binding.ChicleRound.from_problem(p, max_solvers=K)
    o = oracle_mod.OracleCoCoA.from_problem(p, l1=l1)
    if l1:
        r.set_l1(l1)
    table = (np.arange(len(bounds) - 1) % K).astype(np.int32)
    r.assign(K, table)
    o.assign(K, table)
    # (None: rows that share so much that the solver goes row by row, which the private vectors are merged after)
    print(r.debug_solver(), r.debug_passes(), flush=True)
    assert r.debug_passes()[0] == dots
    assert r.debug_solver()[0] == "rowwise" if merge is None else r.debug_solver()[0] == "blocks" and r.debug_passes()[1] == merge
    for k in range(4):
        if by_name:
            r.set_solver("rowwise" if k == 1 else "auto")
        perms = [g.permutation(m).astype(np.int32) for m in o.rows_per_solver()]
        floor = dw_floor(float(np.linalg.norm(o.w)))
        r.local_epoch(r.upload_perm(perms))
        dws = o.local_epoch(perms)
        if k != 2:                                    # (a merge with and without a read-out before it)
            for s in range(K):
                err = rel_l2(r.get_delta_w(s), dws[s], floor)
                assert err <= TOL_DW, (k, s, err)
        o.aggregate()
        r.aggregate()
        P, D, G = r.gap()
        Po, Do, Go = o.gap()[:3]
        err = rel_l2(r.get_w(), o.w, 1e-30)
        print("round %d w %.2e primal %.2e dual %.2e" % (k, err, abs(P - Po) / abs(Po), abs(D - Do) / max(abs(Do), 1e-30)), flush=True)
        # the float mirror rounds w by 2^-24 of its entries; the updates' own errors, a few 2^-24 of each, come on top
        assert err <= 1e-6
        assert abs(P - Po) <= 1e-6 * abs(Po) and abs(G - Go) <= gap_tolerance(Go, Po)
    r.close()


def test_many_blocks_of_rows_use_the_whole_chip():
    """34 blocks of rows leave a block fewer parts than there are L2 partitions: the parts are dealt out over all of these."""
    import paper_1909_04885_amd as binding
    n, m, d = 33 * 16384 + 129, 97, 1500000
    print("\ncase column blocks n=%d m=%d d=%d" % (n, m, d), flush=True)
    g = np.random.default_rng(5)
    step = g.integers(1, d // m, n).astype(np.int32)
    col = (g.integers(0, d, n) % (d - step * (m - 1))).astype(np.int32)[:, None] + step[:, None] * np.arange(m, dtype=np.int32)
    val = (g.random((n, m), dtype=np.float32) - np.float32(0.5)) / 5
    y = np.where(g.random(n) < 0.5, -1, 1).astype(np.float32)
    bounds = np.append(np.arange(0, n, 70001), n)
    r = binding.ChicleRound("hinge", n, d, 1.0 / n, len(bounds) - 1, 1, False, n * m)
    for c, (b, e) in enumerate(zip(bounds[:-1], bounds[1:])):
        r.load_chunk_csr(c, m * np.arange(e - b + 1, dtype=np.int32), col[b:e].reshape(-1), val[b:e].reshape(-1), y[b:e])
    r.assign(1, np.zeros(len(bounds) - 1, dtype=np.int32))
    by_column, _, parts, partitions = r.debug_passes()
    assert by_column and 1 < parts < 8 and partitions == 8
    w = g.standard_normal(d).astype(np.float32)
    r.set_w(w)
    P, D, _ = r.gap()
    w64, z = w.astype(np.float64), np.empty(n)
    for b, e in zip(bounds[:-1], bounds[1:]):
        z[b:e] = np.einsum("ij,ij->i", val[b:e].astype(np.float64), w64[col[b:e]])
    ref = 0.5 * (w64 @ w64) / n + np.maximum(0, 1 - y * z).mean()
    print("primal %.3e dual %.3e" % (abs(P - ref) / ref, abs(D + 0.5 * (w64 @ w64) / n) / ref), flush=True)
    # w is exact in a float here, products and sums are in double: what is left is the rounding of m + n additions
    assert abs(P - ref) <= 2.0 ** -53 * (n + m) * ref and abs(D + 0.5 * (w64 @ w64) / n) <= 2.0 ** -53 * d * ref
    r.close()


@pytest.mark.parametrize("n,length,d,loss,by_column", [
    (1000, 115, 20000, "hinge", False), (16000, 115, 20000, "hinge", False), (16000, 115, 20000, "squared", False), (60000, 115, 10000, "hinge", False),
    (60000, 115, 10000, "logistic", True), (1500, 370, 200003, "hinge", True), (16000, 115, 4000003, "hinge", True)])
def test_dot_products_go_the_cheaper_way(n, length, d, loss, by_column):
    """Short rows over a shared vector that the caches hold, and few rows: row by row.  Both ways sum in double."""
    import paper_1909_04885_amd as binding
    print("\ncase dots %s n=%d length=%d d=%d" % (loss, n, length, d), flush=True)
    p, g = _uniform(n, length, d, loss, 5, 16)
    r = binding.ChicleRound.from_problem(p, max_solvers=5)
    r.assign(5, np.arange(5, dtype=np.int32))
    assert r.debug_passes()[0] == by_column
    w = g.standard_normal(d).astype(np.float32)
    r.set_w(w)
    P = r.gap()[0]
    w64 = w.astype(np.float64)
    z = (p.val.astype(np.float64).reshape(n, length) * w64[p.col].reshape(n, length)).sum(axis=1)
    y = p.y.astype(np.float64)
    losses = 0.5 * (z - y) ** 2 if loss == "squared" else np.maximum(0, 1 - y * z) if loss == "hinge" else np.logaddexp(0, -y * z)
    ref = 0.5 * p.lam * (w64 @ w64) + losses.mean()
    print("primal %.3e" % (abs(P - ref) / ref), flush=True)
    # w is exact in a float here, products and sums are in double; the terms' log and exp are good to a few units in the last place
    assert abs(P - ref) <= 2.0 ** -53 * (n + d + length + 8) * ref
    r.close()


@pytest.mark.parametrize("n,length,d,K,by_column", [
    (1500, 250, 200003, 7, True), (3000, 300, 5000011, 16, True), (1000, 110, 30000001, 2, False), (40000, 110, 6000007, 3, False),
    (20000, 250, 40009, 4, False), (4000, 310, 20011, 16, False), (10000, 120, 20011, 16, False), (1000, 110, 2000003, 8, False)])
def test_merge_goes_the_cheaper_way(oracle_mod, n, length, d, K, by_column):
    """Many columns or blocks of rows for few entries, few buckets for many, or entries that solvers' rows share: the merge is through the
    private vectors."""
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    print("\ncase merge form n=%d length=%d d=%d K=%d" % (n, length, d, K), flush=True)
    g = np.random.default_rng(n + d)
    col = (np.sort(g.integers(0, d - length, (n, length)), axis=1) + np.arange(length)).astype(np.int32).reshape(-1)
    val = (g.standard_normal(n * length) / np.sqrt(length)).astype(np.float32)
    y = np.where(g.random(n) < 0.5, -1, 1).astype(np.float32)
    bounds = np.linspace(0, n, 2 * K + 1).astype(np.int64)
    p = Problem("form", "hinge", n, d, 20.0 / n, y, bounds, row_ptr=np.arange(n + 1, dtype=np.int64) * length, col=col, val=val)
    r = binding.ChicleRound.from_problem(p, max_solvers=K)
    o = oracle_mod.OracleCoCoA.from_problem(p)
    table = (np.arange(2 * K) % K).astype(np.int32)
    r.assign(K, table)
    o.assign(K, table)
    assert r.debug_solver()[0] == "blocks" and r.debug_passes()[1] == by_column
    for k in range(2):
        perms = [g.permutation(m).astype(np.int32) for m in o.rows_per_solver()]
        r.local_epoch(r.upload_perm(perms))
        o.local_epoch(perms)
        o.aggregate()
        r.aggregate()
        err = rel_l2(r.get_w(), o.w, 1e-30)
        print("round %d w %.2e" % (k, err), flush=True)
        assert err <= 1e-6                            # (as above)
    r.close()


def _uniform(n, length, d, loss, chunks, seed):
    from workloads.generate import Problem
    g = np.random.default_rng(seed)
    col = (np.sort(g.integers(0, d - length, (n, length)), axis=1) + np.arange(length)).astype(np.int32).reshape(-1)
    val = (g.standard_normal(n * length) / np.sqrt(length) * np.repeat(0.5 + 2 * g.random(n), length)).astype(np.float32)
    y = (g.standard_normal(n) if loss == "squared" else np.where(g.random(n) < 0.5, -1, 1)).astype(np.float32)
    return Problem("room", loss, n, d, 3.0 / n, y, np.linspace(0, n, chunks + 1).astype(np.int64), row_ptr=np.arange(n + 1, dtype=np.int64) * length,
                   col=col, val=val), g


def test_updates_without_the_table_of_unshared_entries(oracle_mod):
    """Many shared entries: with the copy there is no room for the table that a solver's update is spread from.  Rows are gone through
    instead, also those that take no step, whose places in the private vectors hold what the merge before took over the columns."""
    import paper_1909_04885_amd as binding
    K = 4
    p, g = _uniform(3000, 400, 300007, "hinge", 2 * K, 11)
    print("\ncase updates row by row", flush=True)
    r = binding.ChicleRound.from_problem(p, max_solvers=K)
    o = oracle_mod.OracleCoCoA.from_problem(p)
    table = (np.arange(2 * K) % K).astype(np.int32)
    r.assign(K, table)
    o.assign(K, table)
    assert r.debug_solver()[0] == "blocks" and r.debug_solver()[3] and r.debug_passes()[:2] == (True, True)
    still = 0
    for k in range(5):
        perms = [g.permutation(m).astype(np.int32) for m in o.rows_per_solver()]
        before, floor = o.alpha.copy(), dw_floor(float(np.linalg.norm(o.w)))
        r.local_epoch(r.upload_perm(perms))
        dws = o.local_epoch(perms)
        still += int((o.alpha == before).sum())
        if k != 1:
            for s in range(K):
                err = rel_l2(r.get_delta_w(s), dws[s], floor)
                assert err <= TOL_DW, (k, s, err)
        o.aggregate()
        r.aggregate()
        assert rel_l2(r.get_w(), o.w, 1e-30) <= 1e-6
        P, _, G = r.gap()
        Po, _, Go = o.gap()[:3]
        assert abs(P - Po) <= 1e-6 * abs(Po) and abs(G - Go) <= gap_tolerance(Go, Po)
    print("steps of zero: %d" % still, flush=True)
    assert 1000 < still < 14000
    r.close()


@pytest.mark.parametrize("loss", ["hinge", "logistic"])
def test_copy_gives_way_to_the_layout_and_comes_back(oracle_mod, loss):
    """Every column in two rows of the one solver: the block solver's layout takes the copy's place.  With two solvers half of the entries
    are shared, and the copy is made again."""
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    n, q = 800, 300
    m, d = 2 * q, n * q
    print("\ncase copy gives way %s" % loss, flush=True)
    g = np.random.default_rng(12)
    i, k = np.arange(n)[:, None], np.arange(q)[None, :]
    col = np.sort(np.concatenate([k * n + i, k * n + (i - 1 - k) % n], axis=1), axis=1).astype(np.int32)
    assert (np.diff(col, axis=1) > 0).all() and (np.bincount(col.reshape(-1), minlength=d) == 2).all()
    val = (g.standard_normal(n * m) / np.sqrt(m)).astype(np.float32)
    y = np.where(g.random(n) < 0.5, -1, 1).astype(np.float32)
    p = Problem("room", loss, n, d, 3.0 / n, y, np.linspace(0, n, 7).astype(np.int64), row_ptr=np.arange(n + 1, dtype=np.int64) * m,
                col=col.reshape(-1), val=val)
    r = binding.ChicleRound.from_problem(p, max_solvers=2)
    o = oracle_mod.OracleCoCoA.from_problem(p)
    for K, copy in ((1, False), (2, True), (1, False)):
        table = (np.arange(6) % K).astype(np.int32)
        r.assign(K, table)
        o.assign(K, table)
        assert r.debug_solver()[0] == "blocks" and r.debug_passes()[0] == copy, (K, r.debug_solver(), r.debug_passes())
        for k in range(2):
            perms = [g.permutation(x).astype(np.int32) for x in o.rows_per_solver()]
            floor = dw_floor(float(np.linalg.norm(o.w)))
            r.local_epoch(r.upload_perm(perms))
            dws = o.local_epoch(perms)
            for s in range(K):
                assert rel_l2(r.get_delta_w(s), dws[s], floor) <= TOL_DW, (K, k, s)
            o.aggregate()
            r.aggregate()
            assert rel_l2(r.get_w(), o.w, 1e-30) <= 1e-6
            P, _, G = r.gap()
            Po, _, Go = o.gap()[:3]
            assert abs(P - Po) <= 1e-6 * abs(Po) and abs(G - Go) <= gap_tolerance(Go, Po)
    r.close()


@pytest.mark.parametrize("then", ["rowwise", "auto"])
def test_failed_pass_leaves_nothing_to_the_next(then):
    """A pass whose launch reports an error (one that an invalid host call before it has left) does not count: the merge after the next
    pass is of that pass's steps alone, whichever way that pass goes."""
    import ctypes
    import paper_1909_04885_amd as binding
    print("\ncase failed pass, then %s" % then, flush=True)
    p, g = _uniform(1500, 250, 200003, "squared", 4, 14)
    r = binding.ChicleRound.from_problem(p, max_solvers=2)
    r.assign(2, np.array([0, 1, 0, 1], dtype=np.int32))
    assert r.debug_solver()[0] == "blocks" and r.debug_passes()[1]
    orders = lambda: r.upload_perm([g.permutation(int(m)).astype(np.int32) for m in r.solver_rows()])
    alphas = lambda: np.concatenate([r.get_alpha(c) for c in range(4)]).astype(np.float64)
    for k in range(2):
        order, next_order = orders(), orders()
        w0 = r.get_w().astype(np.float64)
        r.gap()
        assert binding.load_library().hipSetDevice(ctypes.c_int(9999)) != 0
        with pytest.raises(binding.ChicleError):
            r.local_epoch(order)
        a0 = alphas()
        r.set_solver(then)
        r.local_epoch(next_order)
        r.aggregate()
        r.gap()
        r.set_solver("auto")
        step = np.zeros(p.d)
        np.add.at(step, p.col, np.repeat((alphas() - a0) / (p.lam * p.n), 250) * p.val)
        err = rel_l2(r.get_w() - w0, step, 1e-30)
        print("round %d error %.2e" % (k, err), flush=True)
        # w and alpha are read out as floats: their changes carry 2^-24 of the values, which here are no larger than 50 times them
        assert np.linalg.norm(step) > 0.02 * np.linalg.norm(w0) and err <= 1e-5
    r.close()


@pytest.mark.parametrize("loss", ["hinge", "squared"])
def test_more_buckets_than_are_counted_in_lds(loss):
    """Over 134 million columns: the copy's buckets are counted and filled in memory.  The last column is the last of all buckets."""
    import paper_1909_04885_amd as binding
    n, m, d, K = 240, 900, 16384 * 8192 + 70007, 18
    print("\ncase many buckets %s" % loss, flush=True)
    p, g = _uniform(n, m, d, loss, 2 * K, 15)
    p.col[m - 1::m] = d - 1 - np.arange(n) % 3        # (columns that several rows of every solver hold, too)
    r = binding.ChicleRound.from_problem(p, max_solvers=K)
    alphas = lambda: np.concatenate([r.get_alpha(c) for c in range(2 * K)]).astype(np.float64)
    held = np.unique(p.col)
    for solvers, by_column in ((K, True), (2, False)):
        r.assign(solvers, (np.arange(2 * K) % solvers).astype(np.int32))
        assert r.debug_solver()[0] == "blocks" and r.debug_passes()[:2] == (True, by_column)
        for k in range(2):
            a0, w0 = alphas(), r.get_w()[held].astype(np.float64)
            r.local_epoch(r.upload_perm([g.permutation(int(x)).astype(np.int32) for x in r.solver_rows()]))
            r.aggregate()
            a, w = alphas(), r.get_w()
            step = np.zeros(len(held))
            np.add.at(step, np.searchsorted(held, p.col), np.repeat((a - a0) * (1 if loss == "squared" else p.y) / (p.lam * n), m) * p.val)
            full, w = np.count_nonzero(w), w[held].astype(np.float64)
            err = rel_l2(w - w0, step, 1e-30)
            z = (p.val.astype(np.float64).reshape(n, m) * w[np.searchsorted(held, p.col)].reshape(n, m)).sum(axis=1)
            losses = 0.5 * (z - p.y) ** 2 if loss == "squared" else np.maximum(0, 1 - p.y * z)
            P, ref = r.gap()[0], 0.5 * p.lam * (w @ w) + losses.mean()
            print("K=%d round %d error %.2e primal %.2e, %d columns" % (solvers, k, err, abs(P - ref) / ref, full), flush=True)
            # w and alpha are read out as floats: their changes carry 2^-24 of the values, which here are no larger than 50 times them
            assert np.linalg.norm(step) > 0.02 * np.linalg.norm(w0) and err <= 1e-5
            assert full <= len(held) and abs(P - ref) <= 1e-6 * ref
    r.close()
