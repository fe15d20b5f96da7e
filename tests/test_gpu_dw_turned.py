"""dW by operands as they stand, turned by the LDS, and by transposed copies (dw_turns in csrc/mq_plan.h): small integers, so that every sum
is exact in fp32 whatever its order.  Columns that end inside a group of 64, tokens that end inside a block of 32, either tile."""
import pytest
import torch

pytestmark = pytest.mark.gpu

SIZES = [  # M, N, K
    (33, 144, 272),        # copies
    (2049, 336, 1392),     # copies, ranges of tokens
    (70, 7040, 7168),      # copies, 256-tiles
    (1001, 272, 9232),     # as they stand: rows of a part of a line
    (1100, 2304, 4160),    # rows of whole lines
    (2050, 1040, 2064),    # ranges of tokens
    (770, 2320, 9232),     # 256-tiles
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
    # dX in the place of X, and of the only gradient where the shapes agree: both are read before it is written
    dX, dW2 = mq.mq_linear_bwd(X.clone(), Q, one, one, dY, lam, (4, 2)[:nr])
    mine = X.clone()
    mq.mq_linear_bwd(mine, Q, one, one, dY, lam, (4, 2)[:nr], dX=mine, dW=dW)
    assert torch.equal(mine, dX) and torch.equal(dW, want) and torch.equal(dW2, want)


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
