"""The decode GEMV in the forms that are compiled twice, held to 128 registers and not (test_plans.py checks that the sizes take
both): one and two row groups, ragged last row blocks, partial last lines, eight and sixteen waves."""
import pytest
import torch

from tests.util import accumulation_allowance, assert_close, bf16_bits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_06786_amd as mq_

    return mq_


CASES = [(4, 4115, 4128, 3), (5, 7169, 3584, 3), (4, 4001, 4128, 3), (16, 4115, 4096, 3), (4, 1003, 8224, 3), (4, 65601, 288, 3),
         (5, 65601, 640, 2), (16, 70001, 320, 2), (4, 14337, 1600, 2), (1, 65601, 544, 6), (4, 72700, 288, 6), (16, 16385, 1056, 6)]


@pytest.mark.parametrize("B,N,K,r", CASES)
def test_both_register_bounds(mq, oracle, B, N, K, r):
    g = torch.Generator().manual_seed(N + K + B)
    q = torch.randint(0, 256, (N, K), generator=g, dtype=torch.uint8)
    a = (torch.rand(N, generator=g) * 1e-3 + 1e-4).to(torch.bfloat16)
    z = (torch.rand(N, generator=g) * 255).to(torch.bfloat16)
    x = torch.randn(B, K, generator=g).to(torch.bfloat16)
    packed = mq.mq_slice(q.cuda(), r, packed=True)
    y = mq.mq_gemv_sliced(x.cuda(), packed, a.cuda(), z.cuda(), r, K)
    want = oracle.gemv_sliced(bf16_bits(x), packed.cpu().numpy(), bf16_bits(a), bf16_bits(z), r, K)
    assert_close(y.float().cpu().numpy(), want, what=(B, N, K, r),
                 extra=accumulation_allowance(K, 1.0, a.double().numpy() * float(1 << (8 - r)))[None, :])
