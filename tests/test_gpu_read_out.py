"""The read-out of the shared vector around the sizes at which it goes through pinned pieces (2 MiB) and several threads."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, (1 << 20) - 1, 1 << 20, (1 << 20) + 1, 13 * (1 << 19) + 3])
def test_shared_vector_comes_back_as_it_was_set(d):
    import torch
    import paper_1909_04885_amd as binding
    assert torch.cuda.is_available()
    print("\ncase read-out d=%d" % d, flush=True)
    g = binding.ChicleRound("hinge", 4, d, 0.1, 1, 1, False, 4)
    g.load_chunk_csr(0, np.arange(5), np.zeros(4, dtype=np.int32), np.ones(4, dtype=np.float32), np.ones(4, dtype=np.float32))
    g.assign(1, np.zeros(1, dtype=np.int32))
    for seed in range(3):
        w = np.random.default_rng(seed).standard_normal(d).astype(np.float32)
        g.set_w(w)
        assert np.array_equal(g.get_w(), w)
    g.close()


def test_read_out_follows_the_pass_on_a_per_thread_stream():
    """hipStreamPerThread names another stream in every thread: the copies still follow the caller's kernels."""
    import torch
    import paper_1909_04885_amd as binding
    assert torch.cuda.is_available()
    n, d, m = 20000, 3 << 20, 20
    print("\ncase read-out on a per-thread stream d=%d" % d, flush=True)
    rng = np.random.default_rng(2)
    # few columns, so that every pass changes the vector (all at the end of it: the last pieces)
    col = (d - 1 - 50 * m + rng.integers(0, 50, (n, m)) + np.arange(m) * 50).astype(np.int32)
    val = np.full(n * m, 0.2, dtype=np.float32)
    y = np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    with torch.cuda.stream(torch.cuda.ExternalStream(2)):
        g = binding.ChicleRound("hinge", n, d, 1e-4, 1, 1, False, n * m)
    assert g.stream.cuda_stream == 2
    g.load_chunk_csr(0, np.arange(n + 1) * m, col.ravel(), val, y)
    g.assign(1, np.zeros(1, dtype=np.int32))
    g.set_solver("rowwise")                      # tens of milliseconds for the copies to run ahead of
    before = g.get_w()
    for r in range(3):
        g.local_epoch_host_perm(rng.permutation(n))
        g.aggregate()
        w = g.get_w()
        g.sync()
        assert np.array_equal(w, g.get_w())
        assert not np.array_equal(w, before)
        before = w
    g.close()
