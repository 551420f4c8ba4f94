"""Training jobs whose speed is followed: what a program that trains with this package has it do.

A pass is one job on data that is already loaded: a number of CoCoA rounds (local pass of all solvers, merge,
duality gap), with the reassignments of an elastic schedule where there is one, and the model read out at the
end.  A second pass goes on training from where the first one stopped.  The inputs are synthetic, made on the
GPU from the seed, with the shapes and distributions of the workloads in `workloads/`, and they go into the
chunk store through the same loading calls that any program uses.

Results: the shared vector, and the primal and the dual value after every round (the gap is their difference).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1909_04885_amd as chicle

DEVICE = "cuda:0"

# kind        dense: rows of d values; short: sparse rows with Zipf(1.1) column popularity; long: sparse rows with
#             uniform columns
# row_len     entries per sparse row: the median of a log-normal with `spread` (0: every row the same), at most max_len
# solvers     K; `schedule` "round:K ..." changes it (the first entry is the K the job begins with), solvers then
#             being of two speeds, 2 and 1, in turn
# orders      how the visiting orders come: "ahead" (on the GPU, each round announces the next one's), "device"
#             (on the GPU), "host" (a host array each round)
BASE = {"row_len": 0, "spread": 0.0, "max_len": 0, "l1": 0.0, "schedule": ""}


def _case(name, **fields):
    return dict(BASE, name=name, **fields)


def listed():
    return [
        # one round of a very small dense job: launches, waits and the read-out count
        _case("dense_tiny", kind="dense", loss="hinge", n=1000, d=48, lam=1e-3, solvers=4, chunk_rows=256, rounds=1,
              orders="host"),
        # SVM on a small dense set, few solvers
        _case("dense_hinge", kind="dense", loss="hinge", n=4096, d=256, lam=1e-3, solvers=4, chunk_rows=1024, rounds=10,
              orders="device"),
        # wide dense features, odd sizes, logistic regression
        _case("dense_wide", kind="dense", loss="logistic", n=20011, d=1001, lam=1e-4, solvers=8, chunk_rows=1000,
              rounds=3, orders="device"),
        # ridge regression on many short dense rows
        _case("dense_ridge", kind="dense", loss="squared", n=500000, d=28, lam=1e-4, solvers=16, chunk_rows=4096,
              rounds=50, orders="ahead"),
        # small sparse SVM
        _case("sparse_small", kind="short", loss="hinge", n=30000, d=20000, row_len=40, lam=1e-5, solvers=6,
              chunk_rows=1024, rounds=6, orders="device"),
        # sparse SVM of the size the benchmark runs
        _case("sparse_zipf", kind="short", loss="hinge", n=2000000, d=1000000, row_len=40, lam=1e-5, solvers=32,
              chunk_rows=4096, rounds=20, orders="ahead"),
        # sparse logistic regression
        _case("sparse_logistic", kind="short", loss="logistic", n=300000, d=200000, row_len=40, lam=1e-5, solvers=32,
              chunk_rows=4096, rounds=5, orders="ahead"),
        # elastic net, sizes that divide by nothing
        _case("sparse_elastic_net", kind="short", loss="squared", n=100003, d=50021, row_len=33, lam=1e-4, l1=0.05,
              solvers=12, chunk_rows=999, rounds=8, orders="device"),
        # sparse rows of uneven length, as text and click logs have them
        _case("sparse_ragged", kind="short", loss="hinge", n=60007, d=100000, row_len=30, spread=0.6, max_len=200,
              lam=1e-4, solvers=16, chunk_rows=1024, rounds=3, orders="device"),
        # scale-in and scale-out in one job: 32 -> 8 -> 64 -> 16 solvers
        _case("elastic", kind="short", loss="hinge", n=500000, d=400000, row_len=40, lam=1e-5, solvers=32,
              schedule="0:32 5:8 10:64 15:16", chunk_rows=4096, rounds=20, orders="ahead"),
        # small long-row job
        _case("longrow_small", kind="long", loss="hinge", n=1500, d=200000, row_len=300, spread=0.668, max_len=3000,
              lam=1e-6, solvers=7, chunk_rows=128, rounds=4, orders="device"),
        # long hashed rows over many columns, many solvers
        _case("sparse_longrow", kind="long", loss="hinge", n=100000, d=20000000, row_len=800, spread=0.668,
              max_len=20000, lam=1e-6, solvers=64, chunk_rows=1024, rounds=10, orders="device"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another job of the same ranges: any data kind, loss and way of giving orders, sizes spread over their logarithm."""
    kind = rng.choice(["dense", "dense", "short", "short", "short", "long"])
    loss = rng.choice(["hinge", "hinge", "squared", "logistic"])
    c = dict(BASE, kind=kind, loss=loss)
    ragged = False
    if kind == "dense":
        c["d"] = _log_uniform(rng, 8, 1500)
        c["n"] = _log_uniform(rng, 500, min(500000, 14000000 // c["d"]))
    elif kind == "short":
        c["n"] = _log_uniform(rng, 2000, 1500000)
        c["d"] = _log_uniform(rng, 2000, 1000000)
        c["row_len"] = _log_uniform(rng, 10, 44)
        ragged = rng.random() < 0.4
        if ragged:
            c["spread"], c["max_len"] = round(rng.uniform(0.3, 0.7), 3), rng.randint(100, 300)
            c["n"] = min(c["n"], 300000)
    else:
        c["row_len"] = _log_uniform(rng, 150, 1000)
        c["spread"], c["max_len"] = round(rng.uniform(0.3, 0.7), 3), _log_uniform(rng, 2000, 20000)
        c["n"] = _log_uniform(rng, 1000, 60000000 // c["row_len"])
        c["n"] = min(c["n"], 100000)
        c["d"] = _log_uniform(rng, 200000, 20000000)
    n = c["n"]
    c["chunk_rows"] = min(n, max(_log_uniform(rng, 100, 4096), n // 500))
    n_chunks = -(-n // c["chunk_rows"])
    # the shapes that are stepped one row at a time cost microseconds a row, the others far less
    slow = ragged or kind == "long" or (kind == "dense" and c["d"] > 320)
    budget = 15000 if slow else 60000 if loss == "logistic" else 250000
    fewest = max(1, -(-n // budget))
    c["solvers"] = max(fewest, min(_log_uniform(rng, 2, 64), n_chunks))
    c["rounds"] = max(1, min(rng.randint(1, 10), budget * c["solvers"] // n))
    c["lam"] = _log_uniform(rng, 10, 10000) / 100.0 / n       # lambda n between 0.1 and 100
    if rng.random() < 0.15:
        c["l1"] = round(rng.uniform(0.005, 0.05), 4)
    if kind == "short" and n_chunks >= 16 and rng.random() < 0.2:
        c["rounds"] = max(c["rounds"], 4)
        k = max(c["solvers"], min(2 * fewest, n_chunks))
        c["solvers"], c["schedule"] = k, "0:%d %d:%d" % (k, c["rounds"] // 2, max(fewest, k // 2))
    c["orders"] = rng.choice(["ahead", "device", "host"])
    return c


# ---- inputs ---------------------------------------------------------------------------------------------------

def _generator(seed, stream):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(1000003 * int(seed) + stream)
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEVICE, dtype=torch.float64)


def _row_lengths(c, g):
    n = c["n"]
    if not c["spread"]:
        return torch.full((n,), c["row_len"], dtype=torch.int64, device=DEVICE)
    z = torch.randn(n, generator=g, device=DEVICE, dtype=torch.float64)
    return torch.exp(math.log(c["row_len"]) + c["spread"] * z).round().long().clamp(1, min(c["max_len"], c["d"] // 2))


def _labels(c, z, g):
    """Targets from the planted model's margins z: the sign with flips, or the margin with noise."""
    if c["loss"] == "squared":
        return (z + 0.1 * torch.randn(z.numel(), generator=g, device=DEVICE, dtype=torch.float64)).float()
    y = torch.where(z >= 0, 1.0, -1.0)
    return torch.where(_rand(g, z.numel()) < 0.05, -y, y).float()


def _dense(c, seed):
    g = _generator(seed, 1)
    n, d = c["n"], c["d"]
    X = torch.randn(n, d, generator=g, device=DEVICE)
    if c["loss"] != "squared":
        X /= X.square().sum(1, keepdim=True).sqrt()
    w = torch.randn(d, generator=g, device=DEVICE)
    z = (X * w).sum(1, dtype=torch.float64)
    return X, _labels(c, z, g)


def _short_rows(c, seed):
    """Distinct Zipf(1.1) columns per row, popular ones scattered over the ids, values U(0, 1) then normalised."""
    g = _generator(seed, 2)
    n, d = c["n"], c["d"]
    lens = _row_lengths(c, g)
    width = int(lens.max())
    cdf = torch.cumsum(torch.arange(1, d + 1, device=DEVICE, dtype=torch.float64) ** -1.1, 0)

    def ranks(count):
        return torch.searchsorted(cdf, _rand(g, count) * cdf[-1]).clamp(max=d - 1).int()

    place = torch.arange(width, device=DEVICE, dtype=torch.int32)
    rank = torch.empty(n, width, dtype=torch.int32, device=DEVICE)
    for r0 in range(0, n, 1 << 18):
        m = min(n, r0 + (1 << 18)) - r0
        used = place[None, :] < lens[r0:r0 + m, None]
        r = torch.where(used, ranks(m * width).view(m, width), d + place[None, :])   # unused places sort to the end
        r = r.sort(1).values
        todo = torch.arange(m, device=DEVICE)
        while todo.numel():                                                          # columns are distinct in a row
            sub = r[todo]
            dup = torch.zeros_like(sub, dtype=torch.bool)
            dup[:, 1:] = sub[:, 1:] == sub[:, :-1]
            has = dup.any(1)
            todo, sub, dup = todo[has], sub[has], dup[has]
            sub[dup] = ranks(int(dup.sum()))
            r[todo] = sub.sort(1).values
        rank[r0:r0 + m] = r
    ids = torch.randperm(d, generator=g, device=DEVICE).int()
    wide = torch.cat([ids, torch.arange(d, d + width, device=DEVICE, dtype=torch.int32)])
    col = wide[rank.long()].sort(1).values
    used = col < d
    val = torch.rand(n, width, generator=g, device=DEVICE) * used
    val /= val.square().sum(1, keepdim=True).sqrt().clamp(min=1e-6)
    w = torch.zeros(d + width, device=DEVICE)
    support = torch.randperm(d, generator=g, device=DEVICE)[:max(1, d // 100)]
    w[support] = torch.randn(support.numel(), generator=g, device=DEVICE)
    z = (val * w[col.long()]).sum(1, dtype=torch.float64)
    return lens, col[used], val[used], _labels(c, z, g)


def _long_rows(c, seed):
    """Distinct uniform columns, values +-1 / sqrt(row length)."""
    g = _generator(seed, 3)
    n, d = c["n"], c["d"]
    lens = _row_lengths(c, g)
    total = int(lens.sum())
    row = torch.repeat_interleave(torch.arange(n, device=DEVICE), lens)
    key = (row * d + torch.randint(d, (total,), generator=g, device=DEVICE)).sort().values
    while True:
        dup = torch.zeros(total, dtype=torch.bool, device=DEVICE)
        dup[1:] = key[1:] == key[:-1]
        m = int(dup.sum())
        if m == 0:
            break
        key[dup] = key[dup] // d * d + torch.randint(d, (m,), generator=g, device=DEVICE)
        key = key.sort().values
    col = (key - row * d).int()
    sign = 1 - 2 * torch.randint(2, (total,), generator=g, device=DEVICE)
    val = (sign / lens.double()[row].sqrt()).float()
    w = torch.zeros(d, dtype=torch.int64, device=DEVICE)
    support = torch.randperm(d, generator=g, device=DEVICE)[:max(1, d // 100)]
    w[support] = (1000 * torch.randn(support.numel(), generator=g, device=DEVICE)).long()
    z = torch.zeros(n, dtype=torch.int64, device=DEVICE).index_add_(0, row, sign * w[col.long()])   # whole numbers: any order
    return lens, col, val, _labels(c, z.double() / 1000 / lens.double().sqrt(), g)


def _orders(rows, g):
    """A random order of every solver's rows, one solver after the other."""
    rows = torch.as_tensor(rows, device=DEVICE)
    solver = torch.repeat_interleave(torch.arange(rows.numel(), device=DEVICE), rows)
    start = torch.cumsum(rows, 0) - rows
    return ((solver + _rand(g, solver.numel())).argsort(stable=True) - start[solver]).int()


def _schedule(c):
    return {int(r): int(k) for r, k in (item.split(":") for item in c["schedule"].split())} or {0: c["solvers"]}


def prepare(case, seed):
    c = case
    n, d = c["n"], c["d"]
    bounds = list(range(0, n, c["chunk_rows"])) + [n]
    n_chunks = len(bounds) - 1
    schedule = _schedule(c)
    dense = c["kind"] == "dense"
    if dense:
        X, y = _dense(c, seed)
        X, y = X.cpu().numpy(), y.cpu().numpy()
        loads = np.diff(bounds).astype(np.int64) * d
        entries = n * d
    else:
        lens, col, val, y = (_short_rows if c["kind"] == "short" else _long_rows)(c, seed)
        ptr = np.concatenate([[0], np.cumsum(lens.cpu().numpy())])
        col, val, y = col.cpu().numpy(), val.cpu().numpy(), y.cpu().numpy()
        loads = np.diff(ptr[bounds]).astype(np.int64)
        entries = int(ptr[-1])
    torch.cuda.empty_cache()
    g = chicle.ChicleRound(c["loss"], n, d, c["lam"], n_chunks, max(schedule.values()), dense, entries, device=DEVICE)
    for i in range(n_chunks):
        r0, r1 = bounds[i], bounds[i + 1]
        if dense:
            g.load_chunk_dense(i, X[r0:r1], y[r0:r1])
        else:
            p0, p1 = ptr[r0], ptr[r1]
            g.load_chunk_csr(i, ptr[r0:r1 + 1] - p0, col[p0:p1], val[p0:p1], y[r0:r1])
    if c["l1"]:
        g.set_l1(c["l1"])
    elastic = len(schedule) > 1
    gen = _generator(seed, 4)
    orders, rows = [], None
    for r in range(c["rounds"]):
        if r in schedule:
            K = schedule[r]
            g.assign(K, chicle.balance(loads, K, _speeds(K) if elastic else None))
            rows = g.solver_rows()
        order = _orders(rows, gen)
        orders.append(order.cpu().numpy() if c["orders"] == "host" else order)
    g.sync()
    return {"round": g, "case": c, "loads": loads, "orders": orders, "schedule": schedule if elastic else {}}


def _speeds(K):
    return [2 - k % 2 for k in range(K)]


# ---- one pass -------------------------------------------------------------------------------------------------

def run(state):
    g, c, orders, schedule = state["round"], state["case"], state["orders"], state["schedule"]
    rounds = c["rounds"]
    primal, dual = np.empty(rounds), np.empty(rounds)
    announced = False
    for r in range(rounds):
        if r in schedule:
            g.assign(schedule[r], chicle.balance(state["loads"], schedule[r], _speeds(schedule[r])))
        if c["orders"] == "host":
            g.local_epoch_host_perm(orders[r])
        elif c["orders"] == "device":
            g.local_epoch(orders[r])
        else:
            following = orders[r + 1] if r + 1 < rounds and r + 1 not in schedule else None
            g.local_epoch_ahead(None if announced else orders[r], following)
            announced = following is not None
        g.aggregate()
        primal[r], dual[r], _ = g.gap()
    return {"w": g.get_w(), "primal": primal, "dual": dual}


def work(case):
    """Per round: the matrix once for the local pass and once for the gap, the rows' state in both, the private
    vectors written once and merged once, the shared vector; two operations per entry for each of dot product,
    update and gap."""
    c = case
    n, d = c["n"], c["d"]
    dense = c["kind"] == "dense"
    mean = d if dense else min(c["row_len"] * math.exp(c["spread"] ** 2 / 2), c["max_len"] or c["row_len"])
    entries = n * mean
    K = sum(_schedule(c).values()) / len(_schedule(c))
    touched = K * d if dense else min(K * d, entries)
    per_entry = 4 if dense else 8
    per_round = 2 * per_entry * entries + 36 * n + 8 * touched + 20 * d
    return {"bytes": c["rounds"] * per_round, "flops": c["rounds"] * 6 * entries}


def tolerance(case):
    # The state is fp32 (the shared vector is summed in double).  Against the CPU oracle in 64 bits, on the listed
    # and on drawn cases, one and two passes: relative error up to 2.3e-7 (of any of the three outputs), largest
    # single difference 3.1e-6 of the value or the root mean square.
    return {"rel": 1e-6, "max": 1.3e-5}
