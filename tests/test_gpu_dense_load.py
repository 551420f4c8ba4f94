"""Loading dense chunks whose rows are stored longer than they come: every entry arrives, over one part of the device
memory used on the way and over many, and the host holds no second copy of the chunk meanwhile."""
import threading
import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _resident_bytes():
    with open("/proc/self/statm") as f:
        return int(f.read().split()[1]) * 4096


@pytest.mark.parametrize("n,d,solvers", [(1, 1, 1), (3, 5, 1), (130, 27, 2), (70, 4099, 1), (5, 300001, 1), (40, 40961, 64),
                                         (100000, 1001, 4)])
def test_padded_rows_arrive_whole(n, d, solvers):
    import torch
    import paper_1909_04885_amd as binding
    assert torch.cuda.is_available()
    print("\ncase dense load n=%d d=%d" % (n, d), flush=True)
    rng = np.random.default_rng(d)
    X = rng.standard_normal((n, d), dtype=np.float32)
    w = rng.standard_normal(d).astype(np.float32)
    z = np.array([np.dot(x.astype(np.float64), w.astype(np.float64)) for x in X])
    y = (z + 1.0).astype(np.float32)
    lam = 1e-6
    g = binding.ChicleRound("squared", n, d, lam, 1, solvers, True, n * d)
    peak, done, start = [0], threading.Event(), _resident_bytes()

    def watch():
        while not done.is_set():
            peak[0] = max(peak[0], _resident_bytes())
            time.sleep(0.001)
    t = threading.Thread(target=watch)
    t.start()
    g.load_chunk_dense(0, X, y)
    done.set()
    t.join()
    if X.nbytes >= 1 << 28:
        assert peak[0] - start < X.nbytes // 2, "%d MB more while loading %d MB" % ((peak[0] - start) >> 20, X.nbytes >> 20)
    g.assign(1, np.zeros(1, dtype=np.int32))
    # margins and sums are formed in double on both sides; one entry missing or displaced changes its row's margin
    for v in [w] + [np.eye(1, d, k, dtype=np.float32)[0] for k in {0, d // 2, d - 1}]:
        g.set_w(v)
        v = v.astype(np.float64)
        margin = np.array([np.dot(x.astype(np.float64), v) for x in X]) - y
        ref = 0.5 * lam * float(np.dot(v, v)) + 0.5 * float(np.mean(margin ** 2))
        primal = g.gap()[0]
        assert abs(primal - ref) <= 1e-9 * ref, (primal, ref)
    g.close()
