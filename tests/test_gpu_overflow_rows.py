"""The overflow list at the edges of its kernels: row counts around the 16384 counts of a scan step and the 16 of a thread,
rows of one 16-byte chunk, of exactly one wave's chunks and of one more, rows without and full of overflowing codes."""
import numpy as np
import pytest
import torch

from tests.util import first_overflow_code

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_06786_amd as mq_

    return mq_


CASES = [(1, 16, 2), (15, 1024, 4), (17, 1040, 2), (16383, 16, 2), (16384, 32, 3), (16385, 16, 6), (33000, 48, 2), (5, 65536, 2), (3, 64, 8)]


@pytest.mark.parametrize("N,K,r", CASES)
def test_overflow_list(mq, oracle, N, K, r):
    g = torch.Generator().manual_seed(N + K)
    q = torch.randint(0, 256, (N, K), generator=g, dtype=torch.uint8)
    t = first_overflow_code(r)
    q[torch.rand(N, generator=g) < 0.2] = 0                   # rows without a hit
    q[torch.rand(N, generator=g) < 0.1] = min(t, 255)         # every code at the threshold
    q[torch.rand(N, generator=g) < 0.1] = max(t - 1, 0)       # every code just below it
    rp, ci = oracle.overflow_csr(q.numpy(), r)[:2]
    out, ovf = mq.mq_slice(q.cuda(), r, packed=True, extra_precision=True)
    assert np.array_equal(ovf.row_ptr.cpu().numpy(), rp) and int(ovf.nnz) == int(rp[-1])
    assert np.array_equal(ovf.col_idx.cpu().numpy().view(np.uint16)[: int(rp[-1])], ci[: int(rp[-1])])
    # counted in the pass that slices, and cut short by the capacity
    if r in (2, 4):
        cap = max(1, int(rp[-1]) // 2)
        short = mq.Overflow(N, cap)
        short.col_idx.fill_(-1)
        planes, short = mq.mq_slice_multi(q.cuda(), (4, 2), ovf_r=r, ovf=short)
        assert torch.equal(planes[(4, 2).index(r)], out)
        assert np.array_equal(short.row_ptr.cpu().numpy(), rp) and int(short.nnz) == int(rp[-1])
        kept = min(cap, int(rp[-1]))
        assert np.array_equal(short.col_idx.cpu().numpy().view(np.uint16)[:kept], ci[:kept])
