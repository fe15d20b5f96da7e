"""The decode GEMV that forms the sums over the overflow list in its own launch (up to four sequences, 16384 rows and more): ragged
last row blocks, rows of the plane that end inside a line, activations that end inside a staged block, rows without and full of
entries, windows that are continued, and a list that was cut short.  test_plans.py checks which split of the waves each size takes."""
import numpy as np
import pytest
import torch

from tests.util import accumulation_allowance, assert_close, bf16_bits, first_overflow_code

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_06786_amd as mq_

    return mq_


# (six slices of 9216 columns leave too few waves: a launch of its own for the list)
FALLBACK = [(16384, 9216, 2, 3, False)]
IN_ONE_LAUNCH = [
    (16384, 1088, 2, 1, False), (16389, 960, 2, 4, False), (16400, 4608, 2, 2, False), (16400, 4608, 2, 2, True),
    (20000, 2112, 4, 3, False), (18001, 512, 4, 4, True), (36864, 1536, 2, 1, False),
    # one streaming wave; four, whose own part is done before the list's or not, with one to four lines per slice
    (16385, 512, 2, 1, False), (16399, 256, 4, 4, False), (16391, 448, 2, 4, True),
    (16390, 4096, 2, 1, False), (16390, 4096, 2, 3, False), (28677, 4032, 2, 4, False), (16500, 2048, 2, 4, True), (20011, 4096, 4, 3, True),
    (16401, 8192, 2, 1, False), (16397, 6144, 2, 3, False), (33000, 960, 4, 4, False)]


@pytest.mark.parametrize("N,K,r,B,short", IN_ONE_LAUNCH + FALLBACK)
def test_list_in_the_same_launch(mq, oracle, N, K, r, B, short):
    g = torch.Generator().manual_seed(N + K + B)
    t = first_overflow_code(r)
    q = torch.randint(0, t, (N, K), generator=g, dtype=torch.uint8)
    q[torch.rand(N, K, generator=g) < 0.04] = 255
    q[torch.rand(N, generator=g) < 0.01] = 255    # every code of the row overflows
    q[torch.rand(N, generator=g) < 0.05] = 3      # none does
    q[0], q[N - 1] = 255, 255
    a = (torch.rand(N, generator=g) * 1e-3 + 1e-4).to(torch.bfloat16)
    z = (torch.rand(N, generator=g) * 255).to(torch.bfloat16)
    x = torch.randn(B, K, generator=g).to(torch.bfloat16)
    rp, ci = oracle.overflow_csr(q.numpy(), r)[:2]
    cap = int(rp[-1]) // 2 + 1 if short else int(rp[-1])
    packed, ovf = mq.mq_slice(q.cuda(), r, packed=True, extra_precision=True, capacity=cap)
    lists = (np.minimum(rp, cap), ci[:cap])
    y = mq.mq_gemv_sliced(x.cuda(), packed, a.cuda(), z.cuda(), r, K, ovf=ovf)
    want = oracle.gemv_sliced(bf16_bits(x), packed.cpu().numpy(), bf16_bits(a), bf16_bits(z), r, K, ovf=lists)
    assert_close(y.float().cpu().numpy(), want, what=(N, K, r, B, short),
                 extra=accumulation_allowance(K, 1.0, a.double().numpy() * float(1 << (8 - r)))[None, :])
