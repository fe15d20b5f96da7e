"""The decode GEMV with activations in registers on tall planes, on both sides of the rule that chooses how they get there: batches
around twelve, three to five and more slices, ragged last row blocks, int2 and int4."""
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


@pytest.mark.parametrize("N,K,r", [(32773, 512, 2), (32773, 1536, 2), (32768, 2048, 2), (40001, 2560, 2), (32773, 8192, 2), (32773, 1024, 4),
                                   (32773, 768, 4)])
@pytest.mark.parametrize("B", [5, 11, 12, 16])
def test_either_way_to_the_registers(mq, oracle, B, N, K, r):
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
