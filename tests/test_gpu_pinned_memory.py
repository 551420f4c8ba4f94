"""Vectors and visiting orders of up to 1 MB go through pinned memory that kernels read and write: sizes on both sides of that, orders
given again before the last ones are used up, and the error flag, which comes out with the vector or with the gap."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _dense(n, d, seed):
    from workloads.generate import Problem
    g = np.random.default_rng(seed)
    X = g.standard_normal((n, d)).astype(np.float32)
    y = np.where(g.random(n) < 0.5, -1, 1).astype(np.float32)
    return Problem("pinned", "hinge", n, d, 1.0 / n, y, np.array([0, n // 3, n]), X=X), g


@pytest.mark.parametrize("n,d", [(3, 1), (1000, 5), (262143, 4), (262144, 4), (262145, 4)])
def test_orders_from_the_host_without_a_wait_between(n, d):
    import paper_1909_04885_amd as binding
    p, g = _dense(n, d, n)
    print("\ncase pinned orders n=%d" % n, flush=True)
    rounds = [binding.ChicleRound.from_problem(p, max_solvers=2) for _ in range(2)]
    for r in rounds:
        r.assign(2, np.array([0, 1], dtype=np.int32))
    rows = rounds[0].solver_rows()
    for _ in range(4):
        perms = np.concatenate([g.permutation(int(m)) for m in rows]).astype(np.int32)
        keep = perms.copy()
        rounds[0].local_epoch_host_perm(keep)
        keep[:] = 0                                   # (the caller's again)
        rounds[0].aggregate()
        rounds[1].local_epoch(rounds[1].upload_perm(perms))
        rounds[1].aggregate()
    assert np.array_equal(rounds[0].get_w(), rounds[1].get_w())
    assert rounds[0].gap() == rounds[1].gap()
    for r in rounds:
        r.close()


@pytest.mark.parametrize("d", [1, 63, 262143, 262144, 262145])
def test_vector_read_out(d):
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    print("\ncase pinned vector d=%d" % d, flush=True)
    g = np.random.default_rng(d)
    n, m = 200, min(d, 9)
    col = np.concatenate([np.sort(g.choice(d, m, replace=False)) for _ in range(n)]).astype(np.int32)
    p = Problem("pinned", "hinge", n, d, 0.1, np.ones(n, dtype=np.float32), np.array([0, n]),
                row_ptr=np.arange(n + 1, dtype=np.int64) * m, col=col, val=g.random(n * m).astype(np.float32))
    r = binding.ChicleRound.from_problem(p, max_solvers=1)
    r.assign(1, np.zeros(1, dtype=np.int32))
    for _ in range(2):
        w = g.standard_normal(d).astype(np.float32)
        r.set_w(w)
        assert np.array_equal(r.get_w(), w)
    r.close()


@pytest.mark.parametrize("by_gap", [False, True])
def test_refused_order_comes_out_once(by_gap):
    import paper_1909_04885_amd as binding
    p, g = _dense(300, 6, 1)
    r = binding.ChicleRound.from_problem(p, max_solvers=1)
    r.assign(1, np.zeros(2, dtype=np.int32))
    order = g.permutation(300).astype(np.int32)
    order[7] = 300
    r.local_epoch_host_perm(order)
    r.aggregate()
    with pytest.raises(binding.ChicleError):
        r.gap() if by_gap else r.get_w()
    r.get_w()
    r.gap()
    r.close()
