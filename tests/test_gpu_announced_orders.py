"""Announced visiting orders where the solver kind changes between passes: every pass runs with the orders announced last,
also when the pass between used another solver than the one that prepared tiles, or was refused.  Against the oracle."""
import numpy as np
import pytest

from harness import TOL_DW, dw_floor, rel_l2, tail_pairs

pytestmark = pytest.mark.gpu

# solver kind of each pass; "refused": a BATCHED call that the data does not allow, between two passes
SEQUENCES = [["auto", "rowwise", "auto", "auto"], ["auto", "rowwise", "rowwise", "auto", "rowwise", "auto"],
             ["rowwise", "auto", "rowwise_one_cu", "auto"], ["auto", "refused", "auto", "refused", "rowwise", "auto"]]


def _problem(kind, n):
    from workloads.generate import Problem
    g = np.random.default_rng(7)
    y = np.where(g.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    bounds = np.array([0, 70, n // 2 + 34, n], dtype=np.int64)
    if kind != "sparse":
        d = kind
        X = (g.standard_normal((n, d)) / np.sqrt(d)).astype(np.float32)
        return Problem("announced", "hinge", n, d, 0.02, y, bounds, X=X)
    d, m = 600, 20
    col = np.concatenate([np.sort(g.choice(d, m, replace=False)) for _ in range(n)]).astype(np.int32)
    val = (g.standard_normal(n * m) / np.sqrt(m)).astype(np.float32)
    return Problem("announced", "hinge", n, d, 0.02, y, bounds, row_ptr=np.arange(n + 1, dtype=np.int64) * m, col=col, val=val)


@pytest.mark.parametrize("kinds", SEQUENCES, ids=lambda s: "-".join(s))
@pytest.mark.parametrize("kind,short", [(28, False), (100, False), (400, False), (400, True), ("sparse", True)])
def test_pass_runs_the_orders_announced_last(oracle_mod, kind, short, kinds):
    import torch
    import paper_1909_04885_amd as binding
    assert torch.cuda.is_available()
    p = _problem(kind, 333 if kind == "sparse" or short else 2500)     # (short dense passes prepare no tiles)
    print("\ncase announced %s %s" % (kind, kinds), flush=True)
    K, table = 2, np.array([0, 1, 0], dtype=np.int32)
    o = oracle_mod.OracleCoCoA.from_problem(p)
    g = binding.ChicleRound.from_problem(p, max_solvers=K)
    o.assign(K, table)
    g.assign(K, table)
    rng = np.random.default_rng(11)
    perms = [[rng.permutation(int(m)).astype(np.int32) for m in g.solver_rows()] for _ in range(len(kinds) + 1)]
    announced = False
    for r, solver in enumerate(kinds):
        if solver == "refused":
            if kind == 400:           # too wide for the solver by name: refused, and the announcement stands
                g.set_solver("batched")
                with pytest.raises(binding.ChicleError) as e:
                    g.local_epoch_ahead(None, g.upload_perm(perms[0]))
                assert e.value.code == -1
            perms[r + 1] = perms[r]   # the pass that follows runs what is announced already
            continue
        g.set_solver(solver)
        current, following = (None if announced else g.upload_perm(perms[r])), None
        if r + 1 < len(kinds):
            following = g.upload_perm(perms[r + 1])
        g.local_epoch_ahead(current, following)
        announced = following is not None
        floor = dw_floor(float(np.linalg.norm(o.w)))
        ref = o.local_epoch(perms[r])
        for k in range(K):
            e = rel_l2(g.get_delta_w(k), ref[k], floor)
            assert e <= TOL_DW, "pass %d (%s) solver %d: %.3e" % (r, solver, k, e)
        o.aggregate()
        g.aggregate()
    g.close()


# The split batched solver reads pairs of rows beside the tiles, the solver on one compute unit only the tiles: sets formed for
# either are used by the other.
PAIR_SEQUENCES = [["batched_one_cu", "auto"], ["auto", "batched_one_cu", "auto", "batched"],
                  ["batched", "batched_one_cu", "batched_one_cu", "auto", "auto"]]


@pytest.mark.parametrize("kinds", PAIR_SEQUENCES, ids=lambda s: "-".join(s))
def test_tiles_formed_for_the_other_batched_solver(oracle_mod, kinds):
    import torch
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    assert torch.cuda.is_available()
    g = np.random.default_rng(17)
    n, half, d = 2500, 20, 8704 + 9000
    col = np.stack([np.sort(np.concatenate([g.choice(8704, half, replace=False), 8704 + g.choice(9000, half, replace=False)])) for _ in range(n)])
    p = Problem("announced", "hinge", n, d, 1.0 / n, np.where(g.random(n) < 0.5, 1.0, -1.0).astype(np.float32),
                np.array([0, 1200, n], dtype=np.int64), row_ptr=2 * half * np.arange(n + 1, dtype=np.int64),
                col=col.reshape(-1).astype(np.int32), val=(g.standard_normal(col.size) / np.sqrt(2 * half)).astype(np.float32))
    print("\ncase announced pairs %s" % kinds, flush=True)
    K, table = 2, np.arange(2, dtype=np.int32)
    o = oracle_mod.OracleCoCoA.from_problem(p)
    r = binding.ChicleRound.from_problem(p, max_solvers=K)
    o.assign(K, table)
    r.assign(K, table)
    assert r.debug_solver()[:2] == ("batched", 3)
    rows = [np.arange(*p.chunk_rows(k)) for k in range(K)]
    perms = [[g.permutation(x.size) for x in rows] for _ in range(len(kinds) + 1)]
    for order in perms:
        pairs = tail_pairs(p, rows, order)[0]
        assert all(20 < x < 400 for solver in pairs for x in solver[2:-1]), "pairs in every full block, no more than a list holds"
    for i, kind in enumerate(kinds):
        r.set_solver(kind)
        r.local_epoch_ahead(None if i else r.upload_perm(perms[0]), r.upload_perm(perms[i + 1]))
        floor = dw_floor(float(np.linalg.norm(o.w)))
        ref = o.local_epoch(perms[i])
        for k in range(K):
            e = rel_l2(r.get_delta_w(k), ref[k], floor)
            print("pass %d %s solver %d: %.2e" % (i, kind, k, e), flush=True)
            assert e <= TOL_DW, "pass %d (%s) solver %d: %.3e" % (i, kind, k, e)
        o.aggregate()
        r.aggregate()
    r.close()
