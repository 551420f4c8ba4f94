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
