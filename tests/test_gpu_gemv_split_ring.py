"""The K-split decode GEMV at int4 where a wave has fewer weight tiles than its ring has places, exactly as many, and more:
rows from one block of sixteen up to several blocks per wave, one and two lines per slice, a partial last group of slices."""
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


# 256 x K / 8 codes per wave: K = 8192 and 9472 make four and five groups of slices (two lines each, the last group partial);
# K = 6912 has an odd number of lines (one line per slice)
@pytest.mark.parametrize("N,K", [(16, 8192), (40, 9472), (1536, 9472), (4096, 8192), (1000, 6912), (6000, 9472)])
@pytest.mark.parametrize("B", [5, 16])
def test_rings_longer_than_the_work(mq, oracle, B, N, K):
    r = 4
    g = torch.Generator().manual_seed(N + K + B)
    q = torch.randint(0, 256, (N, K), generator=g, dtype=torch.uint8)
    a = (torch.rand(N, generator=g) * 1e-3 + 1e-4).to(torch.bfloat16)
    z = (torch.rand(N, generator=g) * 255).to(torch.bfloat16)
    x = torch.randn(B, K, generator=g).to(torch.bfloat16)
    assert mq.mq_workspace_bytes(mq.MQ_OP_GEMV, B, N, K, r) > 256  # the split form
    packed = mq.mq_slice(q.cuda(), r, packed=True)
    y = mq.mq_gemv_sliced_ws(x.cuda(), packed, a.cuda(), z.cuda(), r, K)
    want = oracle.gemv_sliced(bf16_bits(x), packed.cpu().numpy(), bf16_bits(a), bf16_bits(z), r, K)
    assert_close(y.float().cpu().numpy(), want, what=(N, K, B),
                 extra=accumulation_allowance(K, 1.0, a.double().numpy() * 16.0)[None, :])
