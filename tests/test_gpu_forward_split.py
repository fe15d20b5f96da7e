"""The forward for few tokens (K split over workgroups, a second kernel adds the ranges) at the edges of its tiles: token
blocks of 32, channel tiles of 128, K ranges that are uneven and end inside a 64-wide stage; one to three bit-widths,
extra precision, the gated unit and the objective in its finishing kernel."""
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
    # -- token tiles of one block of 32
    (1, 16, 640, (2,), False),             # one token, an eighth of a channel tile
    (31, 144, 1040, (4,), False),         # K ends 16 into a stage
    (33, 128, 2064, (8,), False),
    (64, 272, 1008, (8, 4, 2), True),
    (77, 528, 4096, (4,), False),
    (97, 80, 3600, (3, 8), False),
    (130, 400, 1616, (8, 4, 2), False),   # two token tiles
    (203, 144, 9216, (2,), True),
    (600, 256, 2304, (6, 2), False),
    # -- two blocks
    (35, 12272, 784, (8,), False),
    (1825, 16, 2720, (2,), False),        # one channel tile, which sums every token block of X itself
    (35, 9280, 544, (4, 8), False),
    (33, 8400, 1552, (8, 4, 2), True),
    # -- three
    (77, 4096, 4096, (4,), False),
    (1218, 144, 2144, (2,), True),        # two channel tiles share three token blocks
    (67, 6576, 528, (4, 2), True),
    (66, 5664, 2192, (4, 3, 2), False),
    # -- four (at two and three bit-widths)
    (116, 8256, 528, (8, 2), False),
    (2038, 16, 29568, (3, 2), True),
    (218, 2704, 4368, (8, 4, 2), False),
]


@pytest.mark.parametrize("M,N,K,rs,ep", CASES)
def test_split_forward(mq, oracle, M, N, K, rs, ep):
    W = _randn(M + N + K, N, K, scale=0.02)
    X = _randn(M * 7 + K, M, K).to(torch.bfloat16)
    Q, a, z = mq.mq_quantize_int8(W.cuda())
    qo, ao, zo = oracle.quantize_int8(W.numpy())
    # the split form is the one that runs: its accumulators are in the workspace
    assert mq.mq_workspace_bytes(mq.MQ_OP_LINEAR_FWD, M, N, K, len(rs)) > 4 * M + 1024
    Y = [torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in rs]
    mq.mq_linear_fwd_multi(X.cuda(), Q, a, z, rs, extra_precision=ep, Y=Y)
    for r, y in zip(rs, Y):
        want = oracle.linear_fwd(bf16_bits(X), qo, ao, zo, r, ep=ep)
        extra = accumulation_allowance(K, 1.0, ao * float(1 << (8 - r)))[None, :]
        assert_close(y.float().cpu().numpy(), want, what=(M, N, K, r), extra=extra)
    # the gated unit and the objective of the finishing kernel: the arithmetic of their stand-alone kernels on the same Y
    GU, A = mq.mq_linear_fwd_multi_gated(X.cuda(), Q, a, z, rs, extra_precision=ep)
    A0 = mq.mq_gated_unit_fwd(Y)
    T = _randn(5, M, N).to(torch.bfloat16).cuda()
    teacher = [-1] + [0] * (len(rs) - 1)
    for mix in (False, True):
        losses, dY = mq.mq_linear_fwd_multi_l2(X.cuda(), Q, a, z, rs, T, teacher, None, mix, extra_precision=ep)
        l0, d0 = mq.mq_matquant_l2_loss(Y, T, teacher, None, mix)
        assert np.allclose(losses.cpu().numpy(), l0.cpu().numpy(), rtol=1e-5)
        for i in range(len(rs)):
            assert torch.equal(dY[i], d0[i]), (rs[i], mix)
    for i in range(len(rs)):
        assert torch.equal(GU[i], Y[i]) and torch.equal(A[i], A0[i]), rs[i]


@pytest.mark.parametrize("M,N,K", [(65, 136, 2048), (66, 5664, 2192), (218, 2704, 4368)])
def test_split_forward_exact(mq, M, N, K):
    """alpha = 1, z = 0 and one-hot activations: every output is one slice value, no rounding anywhere."""
    g = torch.Generator().manual_seed(3)
    q = torch.randint(0, 256, (N, K), generator=g, dtype=torch.int32)
    hot = torch.randint(0, K, (M,), generator=g)
    X = torch.zeros(M, K)
    X[torch.arange(M), hot] = 1.0
    one, nil = torch.ones(N, device="cuda"), torch.zeros(N, device="cuda")
    Y = mq.mq_linear_fwd_multi(X.to(torch.bfloat16).cuda(), q.to(torch.uint8).cuda(), one, nil, (8, 4, 2))
    for r, y in zip((8, 4, 2), Y):
        s = 8 - r
        code = ((q + ((1 << s) >> 1)) >> s).clamp(max=(1 << r) - 1) << s
        assert torch.equal(y.float().cpu(), code[:, hot].t().float()), r


@pytest.mark.parametrize("rs,mix", [((4,), False), ((8, 4, 2), False), ((8, 4, 2), True)])
def test_output_in_the_place_of_the_target(mq, rs, mix):
    """An output may be stored over the target: every element of the target is read before its place is written."""
    M, N, K = 77, 528, 4096
    Q, a, z = mq.mq_quantize_int8(_randn(1, N, K, scale=0.02).cuda())
    X, T = _randn(2, M, K).to(torch.bfloat16).cuda(), _randn(3, M, N).to(torch.bfloat16).cuda()
    teacher = [-1] + [0] * (len(rs) - 1)
    want_l, want = mq.mq_linear_fwd_multi_l2(X, Q, a, z, rs, T, teacher, None, mix)
    Y = mq.mq_linear_fwd_multi(X, Q, a, z, rs)
    over = T.clone()
    losses, dY = mq.mq_linear_fwd_multi_l2(X, Q, a, z, rs, over, teacher, None, mix, Y=[over] + [None] * (len(rs) - 1))
    assert torch.equal(over, Y[0]) and torch.equal(losses, want_l)
    for i in range(len(rs)):
        assert torch.equal(dY[i], want[i]), rs[i]


@pytest.mark.parametrize("M,N,K", [(443, 11472, 4608), (416, 11008, 4096), (77, 4096, 4096)])
def test_objective_at_one_bit_width(mq, M, N, K):
    """The dY of the fused call are those of the two calls in sequence, bit for bit, also where the plain forward takes the
    256-channel tiles that the objective does not have (the first two sizes)."""
    Q, a, z = mq.mq_quantize_int8(_randn(M, N, K, scale=0.02).cuda())
    X, T = _randn(2, M, K).to(torch.bfloat16).cuda(), _randn(3, M, N).to(torch.bfloat16).cuda()
    Y = mq.mq_linear_fwd_multi(X, Q, a, z, (4,))
    _, want = mq.mq_matquant_l2_loss(Y, T)
    _, dY = mq.mq_linear_fwd_multi_l2(X, Q, a, z, (4,), T)
    assert torch.equal(dY[0], want[0])
