"""Every code through the kernels that look r = 2 up instead of computing it (KIND_2 in csrc/mq_linear.h) and through those that do
not: with one-hot inputs, alpha = 1 and z = 0 the outputs are the slices themselves, exactly."""
import pytest
import torch

pytestmark = pytest.mark.gpu

N = K = 256


@pytest.fixture(scope="module")
def mq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_06786_amd as mq_

    return mq_


def _slices(Q, r, ep):
    s = 8 - r
    code = (Q.int() + ((1 << s) >> 1)) >> s
    return ((code if ep else code.clamp(max=(1 << r) - 1)) << s).float()


def _operands(M, repeat):
    n, k = torch.arange(N * repeat).view(-1, 1), torch.arange(K).view(1, -1)
    Q = ((n + 3 * k) % 256).to(torch.uint8).cuda()
    return Q, torch.ones(N * repeat, device="cuda"), torch.zeros(N * repeat, device="cuda")


@pytest.mark.parametrize("ep", [False, True])
@pytest.mark.parametrize("rs", [(2,), (4,), (4, 2), (2, 4), (8, 2), (8, 4, 2), (8, 2, 4), (4, 3, 2)])
@pytest.mark.parametrize("M,repeat", [(20, 1), (77, 9), (300, 1), (1500, 9)])
def test_all_codes(mq, M, repeat, rs, ep):
    Q, alpha, zero = _operands(M, repeat)
    hot = torch.arange(M).cuda()
    X = torch.zeros(M, K, device="cuda", dtype=torch.bfloat16)
    X[hot, hot % K] = 1.0
    Y = mq.mq_linear_fwd_multi(X, Q, alpha, zero, rs, extra_precision=ep)
    for r, y in zip(rs, Y):
        assert torch.equal(y.float(), _slices(Q, r, ep).t()[hot % K]), r
    # backward: one gradient at a time is not zero, and its slice comes out
    for i, r in enumerate(rs):
        dY = [torch.zeros(M, N * repeat, device="cuda", dtype=torch.bfloat16) for _ in rs]
        dY[i][hot, hot % (N * repeat)] = 1.0
        dX, _ = mq.mq_linear_bwd(X, Q, alpha, zero, dY, None, rs, extra_precision=ep, need_dW=False)
        assert torch.equal(dX.float(), _slices(Q, r, ep)[hot % (N * repeat)]), r
