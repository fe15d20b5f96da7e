"""dW by operands as they stand, turned by the LDS, and by transposed copies (dw_turns in csrc/mq_plan.h): small integers, so that every sum
is exact in fp32 whatever its order.  Columns that end inside a group of 64 and inside a tile, tokens that end inside a block of 32,
either tile, whole and in ranges of tokens.  (test_plans.py checks that the sizes take the forms that they are here for.)"""
import pytest
import torch

from tests.util import bf16_bits, rel_l2

pytestmark = pytest.mark.gpu

SIZES = [  # M, N, K
    (33, 144, 272),        # copies
    (840, 224, 288),
    (1041, 160, 304),      # in ranges
    (1028, 2160, 3872),    # 256-tiles
    (1200, 1712, 9424),    # 256-tiles, the last ones in ranges
    (1194, 3376, 160),     # as it stands: a single gradient without dX
    (3329, 160, 1120),     # in ranges
    (1391, 1456, 11168),   # 256-tiles, the last ones in ranges; with dX too
    (1040, 1040, 7264),    # 256-tiles; a summed or scaled gradient in pieces
    (2987, 1232, 3248),    # in ranges
    (1100, 2304, 4160),    # rows of whole lines
    (1286, 2288, 7360),    # of one operand only, in pieces; the last ones in ranges
]


@pytest.fixture(scope="module")
def mq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_06786_amd as mq_

    return mq_


def _ints(seed, *shape):
    return torch.randint(-3, 4, shape, generator=torch.Generator().manual_seed(seed)).to(torch.bfloat16).cuda()


@pytest.mark.parametrize("lam", [None, (0.5, 2.0)])
@pytest.mark.parametrize("nr", [1, 2])
@pytest.mark.parametrize("M,N,K", SIZES)
def test_exact(mq, M, N, K, nr, lam):
    X, dY = _ints(M, M, K), [_ints(7 + i, M, N) for i in range(nr)]
    Q, one = torch.zeros(N, K, dtype=torch.uint8, device="cuda"), torch.ones(N, device="cuda")
    lam = lam and lam[:nr]
    total = sum(d.float() * (lam[i] if lam else 1.0) for i, d in enumerate(dY))
    want = total.t().contiguous() @ X.float()
    _, dW = mq.mq_linear_bwd(X, Q, one, one, dY, lam, (4, 2)[:nr], need_dX=False)
    assert torch.equal(dW, want)
    # dX in the place of X, which is then copied before
    dX, dW2 = mq.mq_linear_bwd(X.clone(), Q, one, one, dY, lam, (4, 2)[:nr])
    mine = X.clone()
    mq.mq_linear_bwd(mine, Q, one, one, dY, lam, (4, 2)[:nr], dX=mine, dW=dW)
    assert torch.equal(mine, dX) and torch.equal(dW, want) and torch.equal(dW2, want)


SQUARE = (1201, 2880)   # tokens, rows and columns


def test_dX_over_the_gradient(mq):
    M, N = SQUARE
    X, dY = _ints(M, M, N), _ints(7, M, N)
    Q, one = torch.zeros(N, N, dtype=torch.uint8, device="cuda"), torch.ones(N, device="cuda")
    want_dX, want = mq.mq_linear_bwd(X, Q, one, one, [dY], None, (4,))
    assert torch.equal(want, dY.float().t().contiguous() @ X.float())
    mine = dY.clone()
    _, dW = mq.mq_linear_bwd(X, Q, one, one, [mine], None, (4,), dX=mine)
    assert torch.equal(dW, want) and torch.equal(mine, want_dX)


CLIP_SIZES = [  # M, N, K: three gradients, one contraction each
    (1115, 1200, 224),
    (1767, 1056, 160),     # in ranges
    (1050, 272, 7280),     # 256-tiles; scaled gradients in pieces
    (3369, 160, 5520),     # in ranges
]


@pytest.mark.parametrize("lam", [None, (0.3, 0.5, 1.0)])
@pytest.mark.parametrize("M,N,K", CLIP_SIZES)
def test_several_gradients(mq, oracle, M, N, K, lam):
    g = torch.Generator().manual_seed(M)
    randn = lambda *shape, scale=1.0: torch.randn(*shape, generator=g) * scale
    W, X, dY = randn(N, K, scale=0.02), randn(M, K).to(torch.bfloat16), [randn(M, N, scale=1e-2).to(torch.bfloat16) for _ in range(3)]
    gamma, beta = torch.rand(N, generator=g) * 0.4 + 0.5, torch.rand(N, generator=g) * 0.4 + 0.5
    Q, a, z = mq.mq_quantize_int8(W.cuda(), gamma.cuda(), beta.cuda())
    got = mq.mq_linear_bwd_clip(W.cuda(), X.cuda(), Q, a, z, [d.cuda() for d in dY], lam, (8, 4, 2), gamma.cuda(), beta.cuda(), want_dalpha_dzero=True)
    want = oracle.clip_factor_grads(W.numpy(), bf16_bits(X), [bf16_bits(d) for d in dY], lam or (1.0,) * 3, (8, 4, 2), gamma.numpy(), beta.numpy())
    for name, mine, ref in zip(("dgamma", "dbeta", "dalpha", "dzero"), got, want):
        # scaled operands are rounded to bf16 once (2^-9.5 rms each), the fp32 sums add next to nothing
        assert rel_l2(mine.cpu().numpy(), ref) <= 1e-2, name


OVER = (1100, 2304, 4160)   # takes operands as they stand


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("nr", [1, 2])
@pytest.mark.parametrize("what", ["X", "dY"])
@pytest.mark.parametrize("first", [0, 2304 * 4160 * 2 - 8])   # from the first element of dW, over its last 16 bytes
def test_dW_over_an_input(mq, what, first, nr, accumulate):
    M, N, K = OVER
    X, dY = _ints(M, M, K), [_ints(7 + i, M, N) for i in range(nr)]
    Q, one = torch.zeros(N, K, dtype=torch.uint8, device="cuda"), torch.ones(N, device="cuda")
    room = torch.zeros(N * K + M * K, device="cuda")
    dW = room[:N * K].view(N, K)
    place = lambda t: room.view(torch.bfloat16)[first:first + t.numel()].view(t.shape).copy_(t)
    inputs = (place(X), dY) if what == "X" else (X, [place(dY[0])] + dY[1:])
    before = dW.clone()   # (with accumulation the bits of the input are what is added to)
    want_dX, want = mq.mq_linear_bwd(X, Q, one, one, dY, None, (4, 2)[:nr], dW=before, accumulate_dW=accumulate)
    dX, _ = mq.mq_linear_bwd(inputs[0], Q, one, one, inputs[1], None, (4, 2)[:nr], dW=dW, accumulate_dW=accumulate)
    assert torch.equal(dW, want) and torch.equal(dX, want_dX)
    if not accumulate:
        assert torch.equal(dW, sum(d.float() for d in dY).t().contiguous() @ X.float())
