"""The forward at three bit-widths with tiles of 64 and 96 tokens, two workgroups to a compute unit: ragged tokens, channels and
contraction, extra precision, without an r = 8 slot, the gated unit and the objective."""
import numpy as np
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


def _randn(seed, *shape, scale=1.0):
    return torch.randn(*shape, generator=torch.Generator().manual_seed(seed)) * scale


CASES = [
    # M, N, K, rs, extra precision
    (700, 2000, 1008, (8, 4, 2), False),    # 64-token tiles
    (450, 2000, 528, (2, 8, 4), True),
    (1300, 1040, 272, (6, 4, 3), False),
    (16, 256, 256, (4, 3, 2), True),        # a quarter of a tile
    (500, 4112, 272, (8, 4, 2), True),      # 96-token tiles
    (2100, 1040, 272, (8, 6, 2), False),
    (450, 12000, 80, (5, 3, 2), False),
]


@pytest.mark.parametrize("M,N,K,rs,ep", CASES)
def test_low_tiles(mq, oracle, M, N, K, rs, ep):
    W = _randn(M + N + K, N, K, scale=0.02)
    X = _randn(M * 7 + K, M, K).to(torch.bfloat16)
    Q, a, z = mq.mq_quantize_int8(W.cuda())
    qo, ao, zo = oracle.quantize_int8(W.numpy())
    Y = [torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in rs]
    mq.mq_linear_fwd_multi(X.cuda(), Q, a, z, rs, extra_precision=ep, Y=Y)
    for r, y in zip(rs, Y):
        want = oracle.linear_fwd(bf16_bits(X), qo, ao, zo, r, ep=ep)
        extra = accumulation_allowance(K, 1.0, ao * float(1 << (8 - r)))[None, :]
        assert_close(y.float().cpu().numpy(), want, what=(M, N, K, r), extra=extra)
    GU, A = mq.mq_linear_fwd_multi_gated(X.cuda(), Q, a, z, rs, extra_precision=ep)
    A0 = mq.mq_gated_unit_fwd(Y)
    T = _randn(5, M, N).to(torch.bfloat16).cuda()
    losses, dY = mq.mq_linear_fwd_multi_l2(X.cuda(), Q, a, z, rs, T, (-1, 0, 0), None, extra_precision=ep)
    l0, d0 = mq.mq_matquant_l2_loss(Y, T, (-1, 0, 0), None)
    assert np.allclose(losses.cpu().numpy(), l0.cpu().numpy(), rtol=1e-5)
    for i in range(len(rs)):
        assert torch.equal(GU[i], Y[i]) and torch.equal(A[i], A0[i]) and torch.equal(dY[i], d0[i]), rs[i]
