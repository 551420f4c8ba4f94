"""Long passes over narrow dense rows, squared loss: the pass as affine maps of runs of rows, at the edges of its row widths,
run lengths and number of solvers, against the oracle at the parity tests' tolerances; its precision, rows that take no step,
announced orders where the solver of the pass changes, the solvers' runtimes."""
import numpy as np
import pytest

from harness import TOL_DW, dw_floor, rel_l2, run_lockstep

pytestmark = pytest.mark.gpu

# 47 blocks of 64 rows are solved block by block, 48 to 191 go in runs of 64 rows (in runs of 128 if all solvers have 4096
# together), up to 399 in runs of 128, more in runs of 256
CASES = [(15, 3073, 1), (16, 12224, 1), (20, 12225, 1), (31, 12289, 1), (28, 25536, 1), (32, 25537, 1), (9, 25700, 2), (2, 3073, 90),
         (1, 3073, 1), (3, 3008, 1), (4, 3100, 1), (5, 4160, 1), (8, 3073, 2), (9, 6200, 3), (16, 3200, 1), (17, 4097, 1),
         (21, 5000, 2), (24, 3073, 1), (28, 16321, 1), (29, 16320, 1), (32, 16449, 1), (32, 3136, 4), (13, 40000, 2)]


@pytest.mark.parametrize("d,n,K", CASES)
def test_affine_runs(oracle_mod, d, n, K):
    """n: rows of the longest solver; the others have a quarter, and one of them none."""
    import torch
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    assert torch.cuda.is_available()
    print("\ncase affine runs n=%d d=%d K=%d" % (n, d, K), flush=True)
    g = np.random.default_rng(100 * d + K)
    sizes = [n // 3, n - n // 3] + [n // 4] * (K - 1 if K < 4 else K - 2)
    bounds = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    total = int(bounds[-1])
    X = (g.standard_normal((total, d)) / np.sqrt(d)).astype(np.float32)
    X[7] = 0                                       # rows that take no step
    X[n - 1] = 0
    y = (X @ g.standard_normal(d) + g.standard_normal(total)).astype(np.float32)
    p = Problem("affine", "squared", total, d, 20.0 / total, y, bounds, X=X)
    table = np.concatenate([[0, 0], np.arange(1, len(sizes) - 1)]).astype(np.int32)
    run_lockstep({"seed": 11, "rounds": 3, "schedule": [(0, K)], "K": K}, p, oracle_mod, binding, check_alpha_every=1, ahead=d % 2 == 0,
                 cancelling=d <= 5, tables=lambda r, Kp, tp: (K, table, table.copy()) if r == 0 else None, max_solvers=K)


def _ridge(n, d, lam_n, seed, unit=True, chunks=2):
    from workloads.generate import Problem
    g = np.random.default_rng(seed)
    X = g.standard_normal((n, d)).astype(np.float32)
    if unit:
        X = (X / np.sqrt(d)).astype(np.float32)
    y = (X @ g.standard_normal(d) / np.sqrt(d) + 0.1 * g.standard_normal(n)).astype(np.float32)
    return Problem("ridge", "squared", n, d, lam_n / n, y, np.linspace(0, n, chunks + 1).astype(np.int64), X=X)


@pytest.mark.parametrize("unit", [False, True])
@pytest.mark.parametrize("lam_n", [0.1, 10.0, 100.0])
@pytest.mark.parametrize("d", [5, 15, 28, 32])
@pytest.mark.parametrize("n", [3500, 26000])
def test_only_what_is_stored_is_rounded(oracle_mod, n, d, lam_n, unit):
    """One pass from zero: the residuals are the targets, exactly.  Alpha is rounded once when it is stored (0.29 of 2^-23 of its
    binade, about 2.5e-8 of the value in the mean square), and so are the update, the squared norms and c, which enter a step
    relative to the whole: about 4.5e-8 together, twice that allowed.  (Maps and dot products in float: alpha 5e-8 to 7e-7,
    updates 3e-8 to 1.5e-7.)"""
    import torch
    import paper_1909_04885_amd as binding
    assert torch.cuda.is_available()
    print("\ncase affine precision n=%d d=%d lambda n=%g %s" % (n, d, lam_n, unit), flush=True)
    p = _ridge(n, d, lam_n, d + n, unit)
    r = binding.ChicleRound.from_problem(p, max_solvers=1)
    o = oracle_mod.OracleCoCoA.from_problem(p)
    table = np.zeros(2, dtype=np.int32)
    r.assign(1, table)
    o.assign(1, table)
    g = np.random.default_rng(d)
    X = p.X.astype(np.float64)
    w_old, drift, rounds = np.zeros(d), 0.0, 12
    for rnd in range(rounds):
        perm = [g.permutation(n).astype(np.int32)]
        r.local_epoch(r.upload_perm(perm))
        ulp = 2.0 ** -24
        if rnd == 0:
            ref = o.local_epoch(perm)[0]
            update = np.linalg.norm(r.get_delta_w(0) - ref) / np.linalg.norm(ref)
        r.aggregate()
        w = r.get_w().astype(np.float64)
        drift += (ulp * np.linalg.norm(w - w_old)) ** 2
        w_old = w
        if rnd not in (0, rounds - 1):
            continue
        a = np.concatenate([r.get_alpha(0), r.get_alpha(1)]).astype(np.float64)
        if rnd == 0:
            alpha = np.linalg.norm(a - o.alpha) / np.linalg.norm(o.alpha)
            print("update %.1e alpha %.1e" % (update, alpha))
            assert update <= 9e-8 and alpha <= 9e-8
        # w against the sum of the alphas' rows: half a unit in the last place of w as it is read, of every update, and in every
        # round of every stored alpha, independently.  (Maps and dot products in float: 4e-7 to 6e-7 of w from the start.)
        stored = (rnd + 1) * (ulp * np.linalg.norm(a[:, None] * X) / lam_n) ** 2
        off = np.linalg.norm(w - X.T @ a / lam_n)
        print("round %d: w off by %.1e, %.1e allowed" % (rnd, off / np.linalg.norm(w), (ulp * np.linalg.norm(w) + 2 * np.sqrt(drift + stored)) / np.linalg.norm(w)))
        assert off <= ulp * np.linalg.norm(w) + 2 * np.sqrt(drift + stored)
    r.close()


@pytest.mark.parametrize("scales", [[1e20, 1e22], [1e-20, 3e-20, 1e-19, 1e-10]], ids=["huge", "tiny"])
@pytest.mark.parametrize("d,n", [(5, 3200), (28, 3200), (32, 13000)])
def test_rows_whose_norm_a_float_can_hardly_hold(d, n, scales):
    """Against row by row: a row beyond a float's range takes no step."""
    import torch
    import paper_1909_04885_amd as binding
    assert torch.cuda.is_available()
    print("\ncase affine extreme rows n=%d d=%d %s" % (n, d, scales), flush=True)
    p = _ridge(n, d, 0.02 * n, 5)
    rows = np.random.default_rng(6).choice(n, 200, replace=False)
    p.X[rows] *= np.resize(scales, 200).astype(np.float32)[:, None]
    got = []
    for solver in ("auto", "rowwise"):
        r = binding.ChicleRound.from_problem(p, max_solvers=1)
        r.assign(1, np.zeros(2, dtype=np.int32))
        r.set_solver(solver)
        g = np.random.default_rng(9)
        for _ in range(2):
            r.local_epoch(r.upload_perm([g.permutation(n).astype(np.int32)]))
            r.aggregate()
        got.append((np.concatenate([r.get_alpha(0), r.get_alpha(1)]), r.get_w()))
        r.close()
    (alpha, w), (alpha_rows, w_rows) = got
    assert np.isfinite(alpha).all() and np.isfinite(w).all()
    huge = np.sum(p.X.astype(np.float64) ** 2, axis=1) > 3.5e38
    assert huge.sum() == (200 if scales[0] > 1 else 0) and (alpha[huge] == 0).all()
    assert np.max(np.abs(alpha - alpha_rows)) <= 5e-4          # the oracle tests' bound for alpha
    assert np.linalg.norm(w - w_rows) <= 1e-4 * np.linalg.norm(w_rows)


@pytest.mark.parametrize("steps", [[1, 2, 1, 1, 2], [2, 2, 1, 2, 2, 1]], ids=str)
def test_announced_orders_across_assignments(oracle_mod, steps):
    """Solvers of 50 blocks (runs of rows) and of 25 (blocks, tiles formed ahead) in turn, with orders announced all the time:
    an assignment drops them, the pass after it has its own."""
    import torch
    import paper_1909_04885_amd as binding
    assert torch.cuda.is_available()
    print("\ncase affine announced %s" % steps, flush=True)
    n, d = 3200, 24
    p = _ridge(n, d, 20.0, 8)
    r = binding.ChicleRound.from_problem(p, max_solvers=2)
    o = oracle_mod.OracleCoCoA.from_problem(p)
    g = np.random.default_rng(4)
    K, following = 0, None
    for s in steps:
        if s != K:
            K = s
            table = (np.arange(2) % K).astype(np.int32)
            r.assign(K, table)
            o.assign(K, table)
            if following is not None:
                with pytest.raises(binding.ChicleError) as e:
                    r.local_epoch_ahead(None, None)
                assert e.value.code == -1
            following = None
        sizes = [int(m) for m in r.solver_rows()]
        perms = following or [g.permutation(m).astype(np.int32) for m in sizes]
        upcoming = [g.permutation(m).astype(np.int32) for m in sizes]
        r.local_epoch_ahead(None if following else r.upload_perm(perms), r.upload_perm(upcoming))
        following = upcoming
        floor = dw_floor(float(np.linalg.norm(o.w)))
        for k, ref in enumerate(o.local_epoch(perms)):
            assert rel_l2(r.get_delta_w(k), ref, floor) <= TOL_DW
        o.aggregate()
        r.aggregate()
    r.close()


@pytest.mark.parametrize("ahead", [False, True])
@pytest.mark.parametrize("d", [20, 24])
def test_many_solvers(oracle_mod, d, ahead):
    """1078 tiles: with orders announced, the first pass goes in runs of rows, and those of more than 20 columns that follow in
    blocks from the tiles formed beside it."""
    import torch
    import paper_1909_04885_amd as binding
    assert torch.cuda.is_available()
    print("\ncase affine many solvers d=%d ahead=%s" % (d, ahead), flush=True)
    K = 22
    p = _ridge(K * 3073, d, 200.0, 13, chunks=K)
    table = np.arange(K, dtype=np.int32)
    run_lockstep({"seed": 2, "rounds": 4, "schedule": [(0, K)], "K": K}, p, oracle_mod, binding, check_alpha_every=1, ahead=ahead,
                 tables=lambda r, Kp, tp: (K, table, table.copy()) if r == 0 else None, max_solvers=K)


def test_solver_runtimes():
    """The chain of a solver's runs is what its clock covers, to the run: 49 runs of 64 rows take less than 56, 14 far less, none
    next to nothing."""
    import torch
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    assert torch.cuda.is_available()
    print("\ncase affine runtimes", flush=True)
    runs = [49, 56, 14]
    bounds = np.concatenate([[0], np.cumsum(64 * np.array(runs))]).astype(np.int64)
    n, d = int(bounds[-1]), 16
    g = np.random.default_rng(1)
    X = g.standard_normal((n, d)).astype(np.float32)
    p = Problem("runtimes", "squared", n, d, 20.0 / n, X[:, 0].copy(), bounds, X=X)
    r = binding.ChicleRound.from_problem(p, max_solvers=4)
    r.assign(4, np.arange(3, dtype=np.int32))
    ms = []
    for _ in range(25):
        r.local_epoch(r.upload_perm([g.permutation(int(m)).astype(np.int32) for m in r.solver_rows()]))
        ms.append(r.solver_ms())
        r.aggregate()
    ms = np.median(ms, axis=0)
    print("solver ms", ms, flush=True)
    assert ms[0] < 0.92 * ms[1] and ms[2] < 0.5 * ms[0] and 0 <= ms[3] < 0.5 * ms[2]
    r.close()


def test_order_entry_out_of_range_is_reported():
    import torch
    import paper_1909_04885_amd as binding
    from workloads.generate import Problem
    assert torch.cuda.is_available()
    g = np.random.default_rng(3)
    n, d = 3200, 8
    X = g.standard_normal((n, d)).astype(np.float32)
    p = Problem("range", "squared", n, d, 0.01, X[:, 0].copy(), np.array([0, n]), X=X)
    r = binding.ChicleRound.from_problem(p, max_solvers=1)
    r.assign(1, np.zeros(1, dtype=np.int32))
    perm = np.arange(n, dtype=np.int32)
    perm[100], perm[3000] = -1, n
    r.local_epoch(r.upload_perm([perm]))
    r.aggregate()
    with pytest.raises(binding.ChicleError):
        r.gap()
    r.close()
