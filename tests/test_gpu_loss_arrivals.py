"""The losses of a forward with the objective on either side of the number of workgroups up to which the last one to arrive finishes them
(kLossArrivals in csrc/mq_plan.h).  (test_plans.py checks that the sizes lie where they are meant to.)"""
import pytest
import torch

pytestmark = pytest.mark.gpu

SIZES = [  # M, N, K, bit-widths; workgroups
    (142, 16, 80, (2,)),          # whole tiles: 1
    (150, 2608, 48, (4, 8, 2)),   # 63
    (187, 4080, 48, (3, 8)),      # 64
    (258, 1600, 48, (4, 2, 8)),   # 65
    (3, 32, 752, (4, 8, 2)),      # K cut: 4
    (1, 1840, 240, (2, 8)),       # 60
    (2, 1952, 48, (4,)),          # 64
    (542, 16, 592, (2, 4, 8)),    # 68
]


@pytest.fixture(scope="module")
def mq():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_06786_amd as mq_

    return mq_


@pytest.mark.parametrize("M,N,K,rs", SIZES)
def test_losses(mq, M, N, K, rs):
    g = torch.Generator(device="cuda").manual_seed(M)
    Q = torch.randint(0, 256, (N, K), generator=g, device="cuda", dtype=torch.uint8)
    X, T = [torch.randn(M, n, generator=g, device="cuda").to(torch.bfloat16) for n in (K, N)]
    alpha, zero = torch.rand(N, generator=g, device="cuda") * 1e-2, torch.rand(N, generator=g, device="cuda") * 255
    Y = [torch.empty(M, N, dtype=torch.bfloat16, device="cuda") for _ in rs]
    ws = torch.full((mq.mq_workspace_bytes(mq.MQ_OP_LINEAR_FWD_L2, M, N, K, len(rs)),), 255, dtype=torch.uint8, device="cuda")
    seen = []
    for _ in range(3):   # the counter and the sums of a call lie where those of the one before did
        losses = torch.full((len(rs),), float("nan"), device="cuda")
        mq.mq_linear_fwd_multi_l2(X, Q, alpha, zero, rs, T, Y=Y, losses=losses, ws=ws)
        seen.append(losses)
    want = torch.stack([(y.double() - T.double()).square().mean() for y in Y])
    # fp32 sums of at most 100 positive terms in a thread and ten more over a workgroup, 2^-24 of the sum for each, then fp64
    assert ((seen[0].double() - want).abs() <= 112 * 2.0 ** -24 * want).all()
    assert torch.equal(seen[1], seen[0]) and torch.equal(seen[2], seen[0])
