"""The block solver for sparse rows of any length at its edges, against the oracle: rows with more segments than
threads, blocks whose entries are joined in parts, solvers of one row and of none, clusters of 1, 2, 4 and 8 workgroups,
data without a single shared column, unshared columns with and without room for the table that streams them, and more
shared columns than eight workgroups hold or rows than there is room to lay out (the row-wise solver's cases).  Every case
states which solver it is to run."""
import numpy as np
import pytest

from harness import run_lockstep

pytestmark = pytest.mark.gpu


def _rows(g, lens, d, zipf):
    if zipf:
        p = (np.arange(d) + 1.0) ** -1.1
        p /= p.sum()
        ids = g.permutation(d)
        return [np.sort(ids[g.choice(d, int(m), replace=False, p=p)]) for m in lens]
    return [np.sort(g.choice(d, int(m), replace=False)) for m in lens]


def _half_shared(g, n, d):
    """48 columns out of 4000 and 48 of the row's own."""
    return [np.sort(np.concatenate([g.choice(4000, 48, replace=False), 4000 + np.arange(48) + 48 * i])) for i in range(n)]


# what runs: (solver, workgroups per solver, private vectors in float, unshared columns row by row)
G1, G2, G4, G8 = [("blocks", k, False, False) for k in (1, 2, 4, 8)]
CASES = {
    # name: (rows, columns, row lengths, Zipf columns, solvers, l1, what runs)
    "ragged": (700, 5000, lambda g, n: np.clip(np.round(g.lognormal(np.log(30), 0.6, n)), 0, 200), True, 3, 0.0, G1),
    "ragged_l1": (500, 5000, lambda g, n: np.clip(np.round(g.lognormal(np.log(30), 0.6, n)), 0, 200), True, 3, 0.02, G1),
    "just_over": (300, 400, lambda g, n: np.where(np.arange(n) == 7, 49, 20), False, 2, 0.0, G1),
    "more_segments_than_threads": (200, 3000, lambda g, n: g.integers(0, 300, n), False, 2, 0.0, G1),
    "joined_in_parts": (4000, 2500, lambda g, n: np.where(np.arange(n) % 97 == 5, 2500, g.integers(150, 300, n)), False, 2, 0.0, G1),
    "joined_in_many_parts": (20000, 2500, lambda g, n: g.integers(700, 900, n), False, 1, 0.0, G1),
    "parts_made_finer": (12000, 360, lambda g, n: np.full(n, 360), False, 2, 0.0, G1),
    "too_long_for_parts": (150, 2500, lambda g, n: g.integers(1000, 2500, n), False, 2, 0.0, ("rowwise", 4, False, False)),
    "nothing_shared": (65, 100000, lambda g, n: np.full(n, 60), False, 5, 0.0, G1),
    # thirteen rows per solver, twelve, and nine and eight of long rows
    "rows_enough": (65, 300, lambda g, n: np.full(n, 60), False, 5, 0.0, G1),
    "few_rows": (60, 300, lambda g, n: np.full(n, 60), False, 5, 0.0, ("rowwise", 1, False, False)),
    "long_rows_enough": (45, 900, lambda g, n: np.full(n, 200), False, 5, 0.0, G1),
    "few_long_rows": (40, 900, lambda g, n: np.full(n, 200), False, 5, 0.0, ("rowwise", 4, False, False)),
    "unshared_row_by_row": (3000, 148000, lambda g, n: np.full(n, 96), None, 2, 0.0, ("blocks", 1, False, True)),
    "two_members": (1600, 30000, lambda g, n: g.integers(60, 150, n), False, 2, 0.0, G2),
    "four_members": (3600, 60000, lambda g, n: g.integers(60, 150, n), False, 2, 0.0, G4),
    "eight_members": (8000, 100000, lambda g, n: g.integers(60, 150, n), False, 2, 0.0, G8),
    "eight_members_in_float": (11800, 170000, lambda g, n: g.integers(60, 150, n), False, 2, 0.0, ("blocks", 8, True, False)),
    "too_many_shared": (2400, 360000, lambda g, n: g.integers(900, 1100, n), False, 2, 0.0, ("rowwise", 4, False, False)),
    "no_room_to_lay_out": (12000, 500, lambda g, n: np.full(n, 90), False, 2, 0.0, ("rowwise", 1, False, False)),
    "room_to_lay_out": (12000, 500, lambda g, n: np.full(n, 80), False, 2, 0.0, G1),
    "no_room_for_eight_members": (12000, 90000, lambda g, n: np.full(n, 80), False, 2, 0.0, ("rowwise", 1, False, False)),
}
LARGE = {"joined_in_many_parts", "parts_made_finer", "no_room_to_lay_out", "room_to_lay_out", "no_room_for_eight_members"}     # one loss, one round


@pytest.mark.parametrize("name,loss", [(n, l) for n in CASES for l in ("hinge", "squared", "logistic") if l == "hinge" or n not in LARGE])
def test_sparse_blocks(oracle_mod, name, loss):
    import torch
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    assert torch.cuda.is_available()
    n, d, lengths, zipf, K, l1, runs = CASES[name]
    g = np.random.default_rng(23)
    lens = np.asarray(lengths(g, n)).astype(np.int64)
    small = n <= 65
    if not small and name != "unshared_row_by_row":
        lens[3] = 0
    cols = _half_shared(g, n, d) if zipf is None else _rows(g, lens, d, zipf)
    if name == "nothing_shared":
        cols = [np.arange(60) * 1000 + i for i in range(n)]
    rp = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(lens, out=rp[1:])
    val = (g.standard_normal(int(rp[-1])) / np.sqrt(np.maximum(np.repeat(lens, lens), 1))).astype(np.float32)
    y = g.standard_normal(n).astype(np.float32) if loss == "squared" else np.where(g.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    if small:
        bounds = np.arange(n + 1, dtype=np.int64)                  # as many rows for every solver
        table = (np.arange(n) % K).astype(np.int32)
    else:
        bounds = np.array([0, 1, n // 2 + 3, n], dtype=np.int64)   # solver 0: one row and the second half
        table = np.array([0, K - 1, 0], dtype=np.int32)
    p = Problem(name, loss, n, d, 0.01, y, bounds, row_ptr=rp, col=np.concatenate(cols).astype(np.int32), val=val)
    print("\ncase blocks %s %s n=%d d=%d entries=%d longest=%d" % (name, loss, n, d, rp[-1], lens.max()), flush=True)
    chosen = binding.ChicleRound.from_problem(p, max_solvers=K)
    chosen.assign(K, table)
    assert chosen.debug_solver() == runs
    chosen.close()
    run_lockstep({"seed": 3, "rounds": 1 if name in LARGE else 3, "schedule": [(0, K)], "K": K}, p, oracle_mod, binding, check_alpha_every=1, l1=l1,
                 ahead=loss == "squared", tables=lambda r, Kp, tp: (K, table, table.copy()) if r == 0 else None, max_solvers=K)


@pytest.mark.parametrize("n,d,m,K,runs", [
    (1024, 180, 180, 4, "blocks"), (1024, 300, 300, 4, "rowwise"), (1024, 1000, 1000, 4, "rowwise"), (1024, 5000, 5000, 8, "rowwise"),
    (512, 20000, 20000, 4, "rowwise"), (1024, 30000, 5000, 4, "rowwise"), (4096, 3000, 3000, 64, "rowwise"),
    (40, 400, 400, 4, "blocks"), (40, 2000, 2000, 4, "rowwise"), (16, 400, 400, 4, "rowwise"),
    # many rows per solver: tiles in parts on the whole chip against the row-wise solver's long chain
    (30000, 4000, 250, 2, "blocks"), (30000, 250, 250, 2, "blocks"), (30000, 250, 250, 64, "rowwise"),
    # one long row among short ones
    (20000, 16000, 30, 4, "blocks")])
def test_tiles_are_joined_in_parts_only_where_that_pays(n, d, m, K, runs):
    import torch
    import paper_1909_04885_amd as binding
    assert torch.cuda.is_available()
    print("\ncase blocks or row by row n=%d d=%d entries per row %d K=%d" % (n, d, m, K), flush=True)
    g = np.random.default_rng(5)
    lens = np.full(n, m)
    if m == 30:
        lens[n // 2] = 15000
    rp = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(lens, out=rp[1:])
    # distinct columns at uneven steps, another start in every row
    col = np.concatenate([np.sort((g.integers(d) + (d // int(l)) * np.arange(l)) % d) for l in lens]).astype(np.int32)
    r = binding.ChicleRound("hinge", n, d, 0.01, K, K, False, int(rp[-1]))
    bounds = np.linspace(0, n, K + 1).astype(np.int64)
    for c in range(K):
        b, e = bounds[c], bounds[c + 1]
        r.load_chunk_csr(c, rp[b:e + 1] - rp[b], col[rp[b]:rp[e]], np.ones(int(rp[e] - rp[b]), dtype=np.float32),
                         np.ones(e - b, dtype=np.float32))
    r.assign(K, np.arange(K, dtype=np.int32))
    assert r.debug_solver()[0] == runs
    r.close()
