"""The forward at one bit-width with 256-channel tiles: each height of the token tile, channel and token tiles that end
early, contractions that end inside a 64-wide stage, extra precision, the gated unit."""
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
    # M, N, K, r, extra precision
    (450, 12000, 272, 4, False),    # 96-token tiles
    (6000, 1040, 144, 2, True),     # 128
    (4096, 2304, 80, 8, False),     # 160
    (2600, 4112, 144, 4, False),    # 192
    (2200, 2896, 272, 3, True),
]


@pytest.mark.parametrize("M,N,K,r,ep", CASES)
def test_wide_forward(mq, oracle, M, N, K, r, ep):
    W = _randn(M + N + K, N, K, scale=0.02)
    X = _randn(M * 7 + K, M, K).to(torch.bfloat16)
    Q, a, z = mq.mq_quantize_int8(W.cuda())
    qo, ao, zo = oracle.quantize_int8(W.numpy())
    Y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    mq.mq_linear_fwd_multi(X.cuda(), Q, a, z, (r,), extra_precision=ep, Y=[Y])
    want = oracle.linear_fwd(bf16_bits(X), qo, ao, zo, r, ep=ep)
    extra = accumulation_allowance(K, 1.0, ao * float(1 << (8 - r)))[None, :]
    assert_close(Y.float().cpu().numpy(), want, what=(M, N, K, r), extra=extra)
    # the sums and the epilogue are those of the other tiles: one bit-width of a call with two is the same, bit for bit
    both = mq.mq_linear_fwd_multi(X.cuda(), Q, a, z, (r, 5), extra_precision=ep)
    GU, A = mq.mq_linear_fwd_multi_gated(X.cuda(), Q, a, z, (r,), extra_precision=ep)
    assert torch.equal(GU[0], Y) and torch.equal(A[0], mq.mq_gated_unit_fwd([Y])[0])
    if M > 2048:  # (below, the two bit-widths may have their contraction cut)
        assert torch.equal(both[0], Y)
