"""The K-split decode GEMV at int4 where a wave has fewer weight tiles than its ring has places, exactly as many, and more:
rows from one block of sixteen up to several blocks per wave, one and two lines per slice, a partial last group of slices, and
rings of six, four and three tiles (test_plans.py checks that the sizes take these forms)."""
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


# A line holds 256 codes and a group four slices.  K = 8192: 32 lines, two to a slice, four groups; 9472: 37 lines, one to a slice, ten
# groups, the last of one slice; 6912: 27 lines, seven groups, the last of three; 9728: 38 lines, two to a slice, five groups, the last of three
RINGS_OF_SIX = [(16, 8192), (40, 9472), (1536, 9472), (4096, 8192), (1000, 6912), (6000, 9472),
                (2600, 6912), (3001, 6912), (3700, 6912), (808, 9728), (1500, 9728), (2441, 9728), (2500, 9728)]
# 97 lines, 25 groups, ten workgroups to a group: 27, 28, 31, 32, 33 and 34 row blocks per wave, for which rings of 6, 4, 4, 3, 3 tiles fit
# and none (another form); two lines to a slice: 29 and 32 row blocks per wave, rings of 4 and 3
LIMITS = [(4313, 24832), (4472, 24832), (4960, 24832), (5113, 24832), (5280, 24832), (5300, 24832), (8190, 28672), (8100, 32768)]
CASES = RINGS_OF_SIX + LIMITS


@pytest.mark.parametrize("N,K", CASES)
@pytest.mark.parametrize("B", [5, 16])
def test_rings_longer_than_the_work(mq, oracle, B, N, K):
    r = 4
    g = torch.Generator().manual_seed(N + K + B)
    q = torch.randint(0, 256, (N, K), generator=g, dtype=torch.uint8)
    a = (torch.rand(N, generator=g) * 1e-3 + 1e-4).to(torch.bfloat16)
    z = (torch.rand(N, generator=g) * 255).to(torch.bfloat16)
    x = torch.randn(B, K, generator=g).to(torch.bfloat16)
    packed = mq.mq_slice(q.cuda(), r, packed=True)
    y = mq.mq_gemv_sliced_ws(x.cuda(), packed, a.cuda(), z.cuda(), r, K)
    want = oracle.gemv_sliced(bf16_bits(x), packed.cpu().numpy(), bf16_bits(a), bf16_bits(z), r, K)
    assert_close(y.float().cpu().numpy(), want, what=(N, K, B),
                 extra=accumulation_allowance(K, 1.0, a.double().numpy() * 16.0)[None, :])
