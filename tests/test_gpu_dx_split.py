"""dX at the sizes where its tiles and the ranges of its contraction can go wrong: every height of the token tile, ranges of
channels that are uneven and end inside a 64-wide stage, one stage per range, a k tile that ends early, one to three
bit-widths, extra precision."""
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
    (1, 64, 16, (4,), False),               # one stage, one token, a sixteenth of a k tile
    (16, 256, 256, (8, 4, 2), False),       # four ranges of one n tile
    (31, 4112, 272, (2,), False),           # 13 ranges; n ends 16 into a stage
    (33, 1040, 528, (3, 8), True),
    (64, 2000, 1008, (8, 4, 2), True),
    (77, 9216, 240, (8,), False),
    (96, 1616, 9216, (4,), True),           # three tiles of one block, few ranges
    (130, 3600, 3600, (8, 4, 2), False),    # five token blocks, the last with two rows
    (250, 2304, 2320, (6, 2), False),       # two blocks
    (400, 896, 3600, (4,), False),          # tiles of one block, no ranges
    (1201, 2000, 1008, (8, 4, 2), False),   # three blocks, several token tiles and ranges
    # the other heights, with ranges and without, where n and k end inside their tiles
    (131, 80, 13392, (3, 8), False),        # two, no ranges
    (1206, 1184, 80, (8, 4, 2), True),      # two
    (259, 80, 14448, (4,), False),          # three, no ranges
    (65, 416, 11248, (4, 3, 2), False),     # three
    (411, 80, 14032, (6, 2), True),         # four, no ranges
    (2037, 4240, 80, (8, 4, 2), False),     # four
    (2042, 7280, 80, (8, 3), True),         # four
    (525, 80, 13248, (8,), False),          # five, no ranges
    (298, 2160, 3104, (6, 2), False),       # five
    (142, 2192, 11968, (2,), False),        # five
]


@pytest.mark.parametrize("M,N,K,rs,ep", CASES)
def test_dx(mq, oracle, M, N, K, rs, ep):
    W = _randn(M + N + K, N, K, scale=0.02)
    X = _randn(M * 7 + K, M, K).to(torch.bfloat16)
    lam = [0.5 + 0.25 * i for i in range(len(rs))]
    dY = [_randn(i + 11, M, N, scale=1e-3).to(torch.bfloat16) for i in range(len(rs))]
    Q, a, z = mq.mq_quantize_int8(W.cuda())
    qo, ao, zo = oracle.quantize_int8(W.numpy())
    dX = torch.full((M, K), float("nan"), dtype=torch.bfloat16, device="cuda")
    mq.mq_linear_bwd(X.cuda(), Q, a, z, [d.cuda() for d in dY], lam, rs, extra_precision=ep, need_dW=False, dX=dX)
    want = oracle.linear_bwd_dx(qo, ao, zo, [bf16_bits(d) for d in dY], lam, rs, ep=ep)
    extra = sum(accumulation_allowance(N, 1e-3, l * float(ao.max()) * float(1 << (8 - r))) for l, r in zip(lam, rs))
    assert_close(dX.float().cpu().numpy(), want, c_rms=2.0 ** -6, what=(M, N, K, rs), extra=extra)


def test_dx_exact(mq):
    """alpha = 1, z = 0 and one gradient entry per token: every dX value is one slice value times a power of two."""
    M, N, K = 65, 2048, 272
    g = torch.Generator().manual_seed(3)
    q = torch.randint(0, 256, (N, K), generator=g, dtype=torch.int32)
    hot = torch.randint(0, N, (M,), generator=g)
    dY = torch.zeros(M, N)
    dY[torch.arange(M), hot] = 0.5
    one, nil = torch.ones(N, device="cuda"), torch.zeros(N, device="cuda")
    X = torch.zeros(M, K, dtype=torch.bfloat16, device="cuda")
    for r in (8, 4, 2):
        dX, _ = mq.mq_linear_bwd(X, q.to(torch.uint8).cuda(), one, nil, [dY.to(torch.bfloat16).cuda()], None, (r,), need_dW=False)
        s = 8 - r
        code = ((q + ((1 << s) >> 1)) >> s).clamp(max=(1 << r) - 1) << s
        assert torch.equal(dX.float().cpu(), code[hot].float() * 0.5), r
