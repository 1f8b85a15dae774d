"""GPU checks of single branches of the launch code and of kernels at the
sizes where they can go wrong (tile edges, remainders, ends of the ranges)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1309_0302_amd import workloads as wl

pytestmark = pytest.mark.gpu


def topk_indices(R, k):
    """Ascending indices of the k largest |R| (ties by index, zeros never)."""
    a = np.abs(R).ravel()
    order = np.lexsort((np.arange(a.size), -a))[:k]
    return np.sort(order[a[order] > 0])


# 32 entries per bitmap word, 1024 words per scan block: one word, one entry
# past a word, one block, one block and one word, several blocks
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (4, 8, 32), (3, 11, 5), (64, 512, 0),
                                   (64, 512, 32768), (65, 505, 1700), (2100, 129, 20000)])
def test_batch_list_in_index_order(m, n, k):
    """godec_batch_get_S returns the list sorted by linear index, with the
    values of the residual the selection used."""
    from paper_1309_0302_amd.binding import GoDecBatch
    rng = np.random.default_rng(m + n)
    X = torch.from_numpy(rng.standard_normal((m, n)).astype(np.float32)).to("cuda:0")
    Y = torch.from_numpy(rng.standard_normal((70, 40)).astype(np.float32)).to("cuda:0")
    b = GoDecBatch([(X, 1, k, 3), (Y, 2, 140, 4)], 1)
    b.step(2)
    for i, kk in ((0, k), (1, 140)):
        idx, val = b.S(i)
        R = b.residual(i).cpu().numpy()
        ref = topk_indices(R, kk)
        assert np.array_equal(idx.cpu().numpy(), ref)
        assert np.array_equal(val.cpu().numpy(), R.ravel()[ref])
    b.step(1)   # the getter leaves the state of the iterations alone
    c = GoDecBatch([(X, 1, k, 3), (Y, 2, 140, 4)], 1)
    c.step(3)
    for i in (0, 1):
        for u, v in zip(b.S(i), c.S(i)):
            assert torch.equal(u, v)
    b.close()
    c.close()
