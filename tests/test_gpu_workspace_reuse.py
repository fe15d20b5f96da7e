"""A workspace that was sized for the largest token count of a program serves its smaller calls too, also where those would
rather cut their contraction and keep partial sums."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_06786_amd as mq_

    return mq_


def _close(a, b, tol):
    a, b = a.double(), b.double()
    assert float((a - b).norm() / b.norm()) <= tol


@pytest.mark.parametrize("most", [4096, 640])
@pytest.mark.parametrize("M", [16, 77, 300])
def test_smaller_calls(mq, M, most):
    N, K, rs = 2304, 1040, (8, 4, 2)
    g = torch.Generator().manual_seed(M)
    W = (torch.randn(N, K, generator=g) * 0.02).cuda()
    X = torch.randn(M, K, generator=g).to(torch.bfloat16).cuda()
    T = torch.randn(M, N, generator=g).to(torch.bfloat16).cuda()
    Q, a, z = mq.mq_quantize_int8(W)
    lend = lambda op, nr: torch.empty(mq.mq_workspace_bytes(op, most, N, K, nr), dtype=torch.uint8, device="cuda")
    # bf16 outputs of the same sums in another order: at most neighbouring values, a few of them (2^-8 / sqrt(3) if all were)
    for bits in (rs, (4,)):
        own = mq.mq_linear_fwd_multi(X, Q, a, z, bits)
        got = mq.mq_linear_fwd_multi(X, Q, a, z, bits, ws=lend(mq.MQ_OP_LINEAR_FWD, len(bits)))
        for x, y in zip(got, own):
            _close(x, y, 2.5e-3)
    losses, dY = mq.mq_linear_fwd_multi_l2(X, Q, a, z, rs, T)
    got, _ = mq.mq_linear_fwd_multi_l2(X, Q, a, z, rs, T, ws=lend(mq.MQ_OP_LINEAR_FWD_L2, 3))
    _close(got, losses, 1e-3)
    dX, dW = mq.mq_linear_bwd(X, Q, a, z, dY, None, rs)
    gX, gW = mq.mq_linear_bwd(X, Q, a, z, dY, None, rs, ws=lend(mq.MQ_OP_LINEAR_BWD, 3))
    _close(gX, dX, 2.5e-3)
    _close(gW, dW, 1e-5)   # fp32 sums of M terms
    ones = torch.ones(N, device="cuda")
    for x, y in zip(mq.mq_linear_bwd_clip(W, X, Q, a, z, dY, None, rs, ones, ones, ws=lend(mq.MQ_OP_LINEAR_BWD_CLIP, 3)),
                    mq.mq_linear_bwd_clip(W, X, Q, a, z, dY, None, rs, ones, ones)):
        _close(x, y, 1e-3)  # sums of mixed sign over K
    short = torch.empty(64, dtype=torch.uint8, device="cuda")
    with pytest.raises(mq.MqError):
        mq.mq_linear_bwd(X, Q, a, z, dY, None, rs, ws=short)
    with pytest.raises(mq.MqError):
        mq.mq_linear_bwd_clip(W, X, Q, a, z, dY, None, rs, ones, ones, ws=short)


@pytest.mark.parametrize("rs", [(8, 4, 2), (3, 8)])
def test_clip_gradients_with_one_matrix(mq, rs):
    """The workspace of one bit-width serves several, one after the other."""
    M, N, K = 300, 272, 1040
    g = torch.Generator().manual_seed(5)
    W = (torch.randn(N, K, generator=g) * 0.02).cuda()
    X = torch.randn(M, K, generator=g).to(torch.bfloat16).cuda()
    dY = [(torch.randn(M, N, generator=g) * 1e-3).to(torch.bfloat16).cuda() for _ in rs]
    gamma, beta = torch.rand(N, generator=g).cuda() * 0.2 + 0.8, torch.rand(N, generator=g).cuda() * 0.2 + 0.8
    Q, a, z = mq.mq_quantize_int8(W, gamma, beta)
    args = W, X, Q, a, z, dY, [0.5 + 0.25 * i for i in range(len(rs))], rs, gamma, beta
    want = mq.mq_linear_bwd_clip(*args, want_dalpha_dzero=True)
    one = mq.mq_workspace_bytes(mq.MQ_OP_LINEAR_BWD_CLIP, M, N, K, 1)
    assert one < mq.mq_workspace_bytes(mq.MQ_OP_LINEAR_BWD_CLIP, M, N, K, len(rs)) - N * K * 4 + 1
    for bytes_ in (one, N * K * 4 + 2 * (N + K) * 320 + 16 * N + 1024):   # (the second: nothing is cut along the tokens)
        got = mq.mq_linear_bwd_clip(*args, want_dalpha_dzero=True, ws=torch.empty(bytes_, dtype=torch.uint8, device="cuda"))
        for x, y in zip(got, want):
            _close(x, y, 1e-5)   # fp32 sums of M terms in another order
    with pytest.raises(mq.MqError):
        mq.mq_linear_bwd_clip(*args, ws=torch.empty(N * K * 4, dtype=torch.uint8, device="cuda"))
