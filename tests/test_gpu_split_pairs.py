"""Two tail workgroups per solver, whose gathers leave out the three latest blocks: what blocks b - 2 and b - 3 add comes through
pairs of rows.  Solvers of one to a few blocks behind a longer one that holds the same columns, tiles in runs, blocks of hundreds
of pairs and of more than a list holds (foreseen from the columns' popularity or not), against the oracle.  Orders of all passes
but the first are announced: their pairs are listed whatever the loss."""
import numpy as np
import pytest

from harness import TOL_DW, dw_floor, gap_tolerance, rel_l2, tail_pairs

pytestmark = pytest.mark.gpu


def _uniform(g, n, d, m):
    return [np.sort(g.choice(d, m, replace=False)) for _ in range(n)], [g.permutation(n) for _ in range(2)]


def _even(g, n, d, m):
    """Every column in as many rows as any other."""
    width = d // m
    return list(np.stack([q * width + g.permutation(n) % width for q in range(m)], axis=1)), [g.permutation(n) for _ in range(2)]


def _groups(g, n, size=8):
    """24 popular columns and 24 that `size` rows hold in common; half of a group two blocks behind the other half."""
    d = 9000 + 24 * (-(-n // size))
    cols = [np.sort(np.concatenate([g.choice(9000, 24, replace=False), 9000 + 24 * (i // size) + np.arange(24)])) for i in range(n)]
    orders = []
    for _ in range(2):
        sets = np.array_split(g.permutation(-(-n // size)), max(1, n // 256))
        order = []
        for s in sets:                       # four blocks: first halves in two of them, second halves in the other two
            rows = [np.arange(size * k, min(n, size * k + size)) for k in s]
            order += [np.concatenate([r[:size // 2] for r in rows]), np.concatenate([r[size // 2:] for r in rows])]
        orders.append(np.concatenate(order))
    return d, cols, orders


def _shared(g, solver_rows, n_tail, holders, filler=0, n_popular=8640):
    """Rows of 44 entries: n_tail in unpopular columns, twelve of them in columns of `holders` rows each, the rest in columns of
    the row's own; popular columns otherwise.  `filler` rows of popular columns come first and make those the more frequent
    ones."""
    n = sum(solver_rows)
    m_pop = 44 - n_tail
    pop = (np.arange((n + filler) * 44, dtype=np.int64) * 7 % n_popular).reshape(-1, 44)
    groups = max(1, -(-n // holders))
    shared = np.stack([n_popular + q * groups + g.permutation(n) % groups for q in range(12)], axis=1)
    own = n_popular + 12 * groups + np.arange(n * (n_tail - 12)).reshape(n, n_tail - 12)
    cols = [np.sort(c) for c in pop[:filler]] + list(np.sort(np.concatenate([pop[filler:, :m_pop], shared, own], axis=1), axis=1))
    return n_popular + 12 * groups + max(1, n * (n_tail - 12)), cols


def _problem(g, name, loss, d, cols, bounds):
    from workloads.generate import Problem
    rp = np.concatenate([[0], np.cumsum([c.size for c in cols])]).astype(np.int64)
    col = np.concatenate(cols).astype(np.int32)
    n = len(cols)
    y = (np.where(g.random(n) < 0.5, -1.0, 1.0) if loss != "squared" else g.standard_normal(n)).astype(np.float32)
    return Problem(name, loss, n, d, 1.0 / n, y, np.asarray(bounds, dtype=np.int64), row_ptr=rp, col=col,
                   val=(g.standard_normal(col.size) / 7.0).astype(np.float32))


def _run(oracle_mod, p, K, table, passes, workgroups=3):
    """The passes against the oracle, each announcing the next one's orders."""
    import paper_1909_04885_amd as binding
    o, r = oracle_mod.OracleCoCoA.from_problem(p), binding.ChicleRound.from_problem(p, max_solvers=K)
    o.assign(K, table)
    r.assign(K, table)
    assert r.debug_solver()[:2] == ("batched", workgroups)
    for i, orders in enumerate(passes):
        r.local_epoch_ahead(None if i else r.upload_perm(orders), r.upload_perm(passes[i + 1]) if i + 1 < len(passes) else None)
        floor = dw_floor(float(np.linalg.norm(o.w)))
        for k, ref in enumerate(o.local_epoch(orders)):
            e = rel_l2(r.get_delta_w(k), ref, floor)
            print("pass %d solver %d update %.2e" % (i, k, e), flush=True)
            assert e <= TOL_DW
        o.aggregate()
        r.aggregate()
        got, want = r.gap(), o.gap()
        assert abs(got[2] - want[2]) <= gap_tolerance(want[2], want[0])
    r.close()


@pytest.mark.parametrize("n_tail", [12, 30])             # the last 24 entries of a row cover its unpopular columns, and not
@pytest.mark.parametrize("n", [1, 64, 65, 128, 129, 192, 193, 256, 257, 321, 449])
def test_few_blocks(oracle_mod, n, n_tail):
    """Two solvers of n rows behind one of 2048, whose last 192 visited rows are in the same unpopular columns: what must not be
    paired across solvers would show."""
    import torch
    assert torch.cuda.is_available()
    print("\ncase few blocks n=%d tails of %d" % (n, n_tail), flush=True)
    g = np.random.default_rng(31)
    filler, extra = 1856, 192
    d, cols = _shared(g, [extra, n, n], n_tail, 3, filler)
    p = _problem(g, "few", "hinge" if n % 2 else "squared", d, cols, [0, filler + extra, filler + extra + n, filler + extra + 2 * n])
    rows = [np.arange(*p.chunk_rows(k)) for k in range(3)]
    passes = [[np.concatenate([g.permutation(filler), filler + g.permutation(extra)]), g.permutation(n), g.permutation(n)] for _ in range(3)]
    for orders in passes:
        pairs, longest = tail_pairs(p, rows, orders)
        assert (longest <= 24) == (n_tail <= 24) and max(max(x) for x in pairs) <= 512
        assert (sum(pairs[1]) + sum(pairs[2]) > 0) == (n > 128)
    _run(oracle_mod, p, 3, np.arange(3, dtype=np.int32), passes)


@pytest.mark.parametrize("n_tail", [12, 30])
def test_tiles_in_runs(oracle_mod, n_tail):
    """Some 2200 tiles of five solvers: runs of five tiles to a workgroup, solvers that begin inside a run."""
    import torch
    assert torch.cuda.is_available()
    print("\ncase tiles in runs, tails of %d" % n_tail, flush=True)
    g = np.random.default_rng(37)
    sizes = [40000, 29017, 30011, 25001, 16064]
    d, cols = _shared(g, sizes, n_tail, 120)
    p = _problem(g, "runs", "hinge", d, cols, np.concatenate([[0], np.cumsum(sizes)]))
    passes = [[g.permutation(x) for x in sizes] for _ in range(2)]
    pairs, longest = tail_pairs(p, [np.arange(*p.chunk_rows(k)) for k in range(5)], passes[1])
    assert (longest <= 24) == (n_tail <= 24) and all(20 < x <= 512 for solver in pairs for x in solver[3:-1])
    _run(oracle_mod, p, 5, np.arange(5, dtype=np.int32), passes)


CASES = [(name, n, loss) for name, n in (("sets", 4000), ("not_listed", 4320), ("too_many", 4133)) for loss in ("hinge", "squared", "logistic")]


@pytest.mark.parametrize("name,n,loss", CASES)
def test_pairs(oracle_mod, name, n, loss):
    import torch
    assert torch.cuda.is_available()
    print("\ncase pairs %s n=%d %s" % (name, n, loss), flush=True)
    g = np.random.default_rng(31)
    if name == "too_many":
        d, cols, orders = _groups(g, n)
    elif name == "not_listed":
        d = 48 * 360                         # (half of the columns unpopular: as many pairs as uniform columns can give)
        cols, orders = _even(g, n, d, 48)
    else:
        d = 16400
        cols, orders = _uniform(g, n, d, 40)
    p = _problem(g, name, loss, d, cols, [0, n])
    most = max(max(tail_pairs(p, [np.arange(n)], [order])[0][0]) for order in orders)
    share = np.sort(np.bincount(p.col, minlength=d))[:max(0, d - 8704)] / n
    expected = 2 * 64 * 64 * float(share @ share)          # pairs of a block, were the rows in random order
    assert {"sets": 100 < most <= 512 and expected < 0.85 * 512, "not_listed": expected > 0.85 * 512,
            "too_many": most > 512 and expected < 0.85 * 512}[name]
    # (two solvers, one of which has no rows, unless all rows are to be in one)
    K = 1 if name == "too_many" else 2
    _run(oracle_mod, p, K, np.zeros(1, dtype=np.int32), [[order] + [np.empty(0, dtype=np.int64)] * (K - 1) for order in orders])


def test_pairs_in_a_context_made_for_long_rows(oracle_mod):
    """Room announced for 120 entries a row, rows of 44: the lists take the place of the long rows' layout."""
    import torch
    import paper_1909_04885_amd as binding
    assert torch.cuda.is_available()
    print("\ncase pairs in a context made for long rows", flush=True)
    g = np.random.default_rng(41)
    n, K = 4000, 2
    d, cols = _shared(g, [n], 12, 10)
    p = _problem(g, "announced_longer", "squared", d, cols, [0, n // 2, n])
    o = oracle_mod.OracleCoCoA.from_problem(p)
    r = binding.ChicleRound(p.loss, n, d, p.lam, K, K, False, 120 * n)
    for k in range(K):
        a, b = p.chunk_rows(k)
        r.load_chunk_csr(k, p.row_ptr[a:b + 1] - p.row_ptr[a], p.col[p.row_ptr[a]:p.row_ptr[b]], p.val[p.row_ptr[a]:p.row_ptr[b]], p.y[a:b])
    table = np.arange(K, dtype=np.int32)
    o.assign(K, table)
    r.assign(K, table)
    assert r.debug_solver()[:2] == ("batched", 3)
    rows = [np.arange(*p.chunk_rows(k)) for k in range(K)]
    perms = [[g.permutation(n // K) for _ in range(K)] for _ in range(3)]
    assert all(x > 50 for order in perms for solver in tail_pairs(p, rows, order)[0] for x in solver[3:-1])
    for i in range(2):
        r.local_epoch_ahead(None if i else r.upload_perm(perms[0]), r.upload_perm(perms[i + 1]))
        ref = o.local_epoch(perms[i])
        for k in range(K):
            assert rel_l2(r.get_delta_w(k), ref[k], dw_floor(float(np.linalg.norm(o.w)))) <= TOL_DW
        o.aggregate()
        r.aggregate()
    r.close()


@pytest.mark.parametrize("loss", ["hinge", "squared", "logistic"])
@pytest.mark.parametrize("n", [65, 3000, 320000])
def test_all_columns_in_the_head(oracle_mod, n, loss):
    """No tails: rows resolved by a wavefront of their own, and beside a tile where tiles and entries are too many for the
    caches (320000 rows; with the logistic loss always).  Rows of 1 to 48 entries, some without any."""
    import torch
    assert torch.cuda.is_available()
    print("\ncase all columns in the head n=%d %s" % (n, loss), flush=True)
    g = np.random.default_rng(43)
    m, d, K = 48, 48 * 40, 3 if n < 1000 else 20
    keep = np.arange(m) < g.integers(0, m + 1, n)[:, None]
    col = np.arange(m) * 40 + g.integers(0, 40, (n, m))
    length = keep.sum(axis=1)
    p = _problem(g, "heads", loss, d, np.split(col[keep], np.cumsum(length)[:-1]), np.linspace(0, n, K + 1).astype(np.int64))
    assert (32768 * (n / 64) + 8 * length.sum() > 224e6) == (n > 300000)
    sizes = [int(np.diff(p.chunk_rows(k))[0]) for k in range(K)]
    _run(oracle_mod, p, K, np.arange(K, dtype=np.int32), [[g.permutation(x) for x in sizes] for _ in range(2)], workgroups=1)


def test_short_rows_fit_a_context_made_for_long_rows(oracle_mod):
    """Such a context holds its private vectors in as many floats as it was announced entries: 8397 for each of twelve solvers, of
    which the columns kept on chip take most."""
    import torch
    import paper_1909_04885_amd as binding
    assert torch.cuda.is_available()
    print("\ncase short rows in little room", flush=True)
    g = np.random.default_rng(47)
    n, d, m, K = 1008, 9000, 40, 12
    cols = list(np.sort(np.argsort(g.random((n, 8000)), axis=1)[:, :m], axis=1))
    p = _problem(g, "little_room", "hinge", d, cols, np.arange(K + 1) * (n // K))
    o, r = oracle_mod.OracleCoCoA.from_problem(p), binding.ChicleRound(p.loss, n, d, p.lam, K, K, False, 100000)
    for k in range(K):
        a, b = p.chunk_rows(k)
        r.load_chunk_csr(k, p.row_ptr[a:b + 1] - p.row_ptr[a], p.col[p.row_ptr[a]:p.row_ptr[b]], p.val[p.row_ptr[a]:p.row_ptr[b]], p.y[a:b])
    table = np.arange(K, dtype=np.int32)
    o.assign(K, table)
    r.assign(K, table)
    orders = [g.permutation(n // K) for _ in range(K)]
    r.local_epoch(r.upload_perm(orders))
    for k, ref in enumerate(o.local_epoch(orders)):
        assert rel_l2(r.get_delta_w(k), ref, dw_floor(0.0)) <= TOL_DW
    r.close()
