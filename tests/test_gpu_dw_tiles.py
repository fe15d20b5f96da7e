"""dW at the edges of its tiles: 128 x 128 and 256 x 256 tiles that end early in either direction, token counts that end
inside a block of 32, ranges of tokens that leave partial tiles (with and without whole rounds before them), accumulation,
several gradients against one X.  (test_plans.py checks that the sizes take the forms that they are here for.)"""
import numpy as np
import pytest
import torch

from tests.util import assert_close, bf16_bits, rel_l2

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
    # M, N, K, nr
    (1, 16, 16, 1),
    (31, 112, 144, 2),       # one 128-tile and the start of the next
    (33, 272, 128, 3),
    (64, 2000, 1008, 3),     # ragged on both sides
    (257, 1104, 3200, 1),
    (1201, 256, 256, 3),     # four tiles in ranges of tokens
    (2050, 144, 272, 2),
    (513, 2304, 2320, 1),
    (2048, 1504, 2000, 1),
    (90, 4112, 4096, 1),     # more than a round of either tile
    # 256-tiles that end early in both directions
    (163, 6976, 1744, 2),    # whole
    (3315, 432, 8416, 1),    # all of them in ranges of tokens
    (1475, 1440, 11120, 1),  # a whole round, then tiles in ranges
]


@pytest.mark.parametrize("M,N,K,nr", CASES)
def test_dw(mq, oracle, M, N, K, nr):
    rs, lam = (8, 4, 2)[:nr], [0.5 + 0.25 * i for i in range(nr)]
    X = _randn(M * 7 + K, M, K).to(torch.bfloat16)
    dY = [_randn(i + 11, M, N, scale=1e-3).to(torch.bfloat16) for i in range(nr)]
    dummy = torch.zeros(N, K, dtype=torch.uint8, device="cuda"), torch.ones(N, device="cuda"), torch.zeros(N, device="cuda")
    dW = torch.full((N, K), float("nan"), device="cuda")
    args = X.cuda(), *dummy, [d.cuda() for d in dY], lam, rs
    mq.mq_linear_bwd(*args, need_dX=False, dW=dW)
    want = oracle.linear_bwd_dw(bf16_bits(X), [bf16_bits(d) for d in dY], lam)
    assert_close(dW.cpu().numpy(), want, c_rms=2.0 ** -6, what=(M, N, K))
    # added to what is there: fp32, one rounding of the sum
    base = _randn(3, N, K, scale=float(np.abs(want).mean())).cuda()
    acc = base.clone()
    mq.mq_linear_bwd(*args, need_dX=False, dW=acc, accumulate_dW=True)
    assert torch.equal(acc, base + dW)


def test_dw_exact(mq):
    """Small integers: every sum is exact in fp32, whatever the order of the tokens."""
    M, N, K = 1500, 400, 272
    g = torch.Generator().manual_seed(3)
    X = torch.randint(-4, 5, (M, K), generator=g).float()
    dY = torch.randint(-4, 5, (M, N), generator=g).float()
    one = torch.ones(N, device="cuda")
    _, dW = mq.mq_linear_bwd(X.to(torch.bfloat16).cuda(), torch.zeros(N, K, dtype=torch.uint8, device="cuda"), one, one,
                             [dY.to(torch.bfloat16).cuda()], None, (4,), need_dX=False)
    assert torch.equal(dW.cpu(), dY.t() @ X)


CLIP_CASES = [
    # M, N, K, rs: one contraction per bit-width, the tiles of all of them dealt together
    (1201, 272, 144, (8, 4, 2)),     # 128-tiles in ranges
    (161, 5712, 720, (8, 4, 2)),     # 256-tiles, whole
    (3144, 5456, 160, (8, 4, 2)),    # 256-tiles in ranges, 22 per gradient
    (1771, 11344, 400, (3, 8, 2)),   # a whole round of 256-tiles, then 14 in ranges
]


@pytest.mark.parametrize("M,N,K,rs", CLIP_CASES)
def test_several_gradients(mq, oracle, M, N, K, rs):
    lam = (0.3, 0.5, 1.0)
    W, X = _randn(M + N, N, K, scale=0.02), _randn(M * 7 + 1, M, K).to(torch.bfloat16)
    dY = [_randn(300 + i, M, N, scale=1e-2).to(torch.bfloat16) for i in range(3)]
    g, b = (torch.rand(N, generator=torch.Generator().manual_seed(i)) * 0.4 + 0.5 for i in (1, 2))
    Q, a, z = mq.mq_quantize_int8(W.cuda(), g.cuda(), b.cuda())
    got = mq.mq_linear_bwd_clip(W.cuda(), X.cuda(), Q, a, z, [d.cuda() for d in dY], lam, rs, g.cuda(), b.cuda(), want_dalpha_dzero=True)
    want = oracle.clip_factor_grads(W.numpy(), bf16_bits(X), [bf16_bits(d) for d in dY], lam, rs, g.numpy(), b.numpy())
    for name, mine, ref in zip(("dgamma", "dbeta", "dalpha", "dzero"), got, want):
        # operands are rounded to bf16 once (2^-9.5 rms each), the fp32 sums add next to nothing
        assert rel_l2(mine.cpu().numpy(), ref) <= 1e-2, name
