"""Rules on sizes (no GPU): what the launches that follow from them rely on."""
import pytest

from tests import (plans, test_gpu_dw_tiles, test_gpu_dw_turned, test_gpu_dx_split, test_gpu_forward_low_tiles, test_gpu_forward_split, test_gpu_forward_wide,
                   test_gpu_gemv_list, test_gpu_gemv_registers, test_gpu_gemv_split_ring, test_gpu_loss_arrivals)

cdiv = lambda a, b: -(-a // b)


@pytest.mark.parametrize("nr", [1, 2, 3])
@pytest.mark.parametrize("K", [16, 512, 896, 4096])
def test_tiles_of_a_forward_fit_one_launch(nr, K):
    """Up to the documented limit of ceil(M / 128) ceil(N / 128) < 2^31 the tiles of the chosen height are below 2^31 too."""
    top = 0x7FFFFF00
    for M, N in [(top, 128 * 127), (128 * 127, top), (46340 * 128, 46340 * 128), (65535 * 128, 32768 * 128), (top, 8), (8192, 14336)]:
        assert cdiv(M, 128) * cdiv(N, 128) < 1 << 31
        p = plans.forward(M, N, K, nr)
        channels = 256 if p.form == "wide" else 128
        assert cdiv(M, 32 * p.blocks) * cdiv(N, channels) < 1 << 31, (M, N, p)


def test_decode_workgroups_share_compute_units():
    """Two workgroups of eight waves share a compute unit at 128 registers only: int3 sizes with more workgroups than compute units
    rely on it wherever their activations leave the LDS for two."""
    seen = set()
    for B in (1, 4, 5, 8, 16):
        for N in range(512, 8192, 176):
            for K in range(256, 12289, 256):
                p = plans.gemv(B, N, K, 3)
                assert p.row_groups == 1
                shared = p.groups > 256 and 2 * p.lds <= 160 * 1024
                if shared:
                    assert p.registers == 128, (B, N, K, p)
                seen.add((shared, p.registers))
    assert seen == {(True, 128), (False, 128), (False, 256)}
    assert [plans.gemv(4, N, K, 3).registers for N, K in ((6000, 4096), (7168, 3584), (4112, 4096), (4000, 2048), (14336, 4096), (73728, 4608))] == [
        128, 128, 128, 256, 256, 256]
    # one workgroup to a compute unit as long as there are no more of them
    assert plans.gemv(4, 14336, 4096, 2).registers == plans.gemv(16, 28672, 4096, 6).registers == plans.gemv(4, 65536, 512, 6).registers == 256
    assert {plans.gemv(B, N, K, r).registers for B, N, K, r in ((4, 14336, 4096, 4), (16, 4096, 4096, 8), (1, 4096, 4096, 2))} == {0}


@pytest.mark.parametrize("B", [5, 16])
def test_split_decode_takes_the_ring_that_fits(B):
    """A shorter ring, and not another form, where six tiles do not fit: up to 33 blocks of 16 rows per wave the split form is taken
    (three tiles: 512 + 24576 + 33 x 4096 bytes of LDS)."""
    for N, K in [(8192, 28672), (7168, 36864), (7680, 30720), (8192, 14080), (4608, 26880), (8192, 14592), (4096, 14336), (4608, 36864)]:
        p = plans.gemv_split(B, N, K, 4)
        assert p.depth == (6 if p.blocks <= 27 else 4 if p.blocks <= 31 else 3) and p.blocks <= 33, (N, K, p)
    seen = set()
    for K in range(6912, 36865, 256):
        for N in range(16, 8193, 112):
            p = plans.gemv_split(B, N, K, 4)
            assert (p.depth > 0) == (p.groups >= 4 and p.blocks <= 33), (N, K, p)
            seen.add(p.depth)
            q = plans.gemv_split(B, N, K, 2)
            assert q.depth == (3 if q.groups >= 4 and q.blocks <= 33 else 0), (N, K, q)
    assert seen == {0, 3, 4, 6}


# ---- the sizes of the GPU tests take the forms that they are there for -------------------------------------------------
def test_split_forward_sizes():
    seen = set()
    for M, N, K, rs, _ in test_gpu_forward_split.CASES:
        p = plans.forward(M, N, K, len(rs))
        assert p.form == "split" and p.ranges > 1, (M, N, K, rs, p)
        seen.add((len(rs), p.blocks))
    assert seen == {(1, 1), (1, 2), (1, 3), (2, 1), (2, 2), (2, 3), (2, 4), (3, 1), (3, 2), (3, 3), (3, 4)}
    # at one bit-width, where the plain forward takes the wide tiles, the objective takes the tiles of the same sums
    assert [plans.forward(M, N, K, 1).form for M, N, K in ((443, 11472, 4608), (416, 11008, 4096), (77, 4096, 4096))] == ["wide", "wide", "split"]


def test_tiled_forward_sizes():
    assert {plans.forward(M, N, K, 3)[:2] for M, N, K, _, _ in test_gpu_forward_low_tiles.CASES} == {("tiled", 2), ("tiled", 3)}
    assert {plans.forward(M, N, K, 1)[:2] for M, N, K, _, _ in test_gpu_forward_wide.CASES} == {("wide", b) for b in (3, 4, 5, 6)}


def test_noalloc_sizes():
    # the comparison with the workspace form is bit for bit: K is not cut there
    assert all(plans.forward(M, N, K, 3).form == "tiled" for M, N, K in ((600, 392, 464), (130, 136, 208)))


def test_dx_sizes():
    seen = {(p.blocks, p.ranges > 1) for p in (plans.dx(M, N, K, len(rs)) for M, N, K, rs, _ in test_gpu_dx_split.CASES)}
    assert seen == {(b, cut) for b in (1, 2, 3, 4, 5) for cut in (False, True)}


def test_dw_sizes():
    form = lambda p: (p.side, p.whole > 0, p.cut > 0)
    seen = {form(plans.dw(M, N, K)) for M, N, K, _ in test_gpu_dw_tiles.CASES}
    assert seen == {(128, True, False), (128, False, True), (256, True, False), (256, False, True), (256, True, True)}
    assert [form(plans.dw(M, N, K, len(rs))) for M, N, K, rs in test_gpu_dw_tiles.CLIP_CASES] == [
        (128, False, True), (256, True, False), (256, False, True), (256, True, True)]
    for M, N, K, rs in test_gpu_dw_tiles.CLIP_CASES:
        assert N % plans.dw(M, N, K, len(rs)).side and K % plans.dw(M, N, K, len(rs)).side


def test_dw_turned_sizes():
    def form(M, N, K, n=1):
        p = plans.dw(M, N, K, n)
        alone, prep = [plans.dw_turns(M, N, K, n, True, p_) for p_ in (False, True)], plans.dw_turns(M, N, K, n, False, True)
        return p.side, p.whole > 0, p.cut > 0, *alone, prep

    # side, whole tiles, tiles in ranges; as they stand: one gradient without dX, with dX, a summed or scaled one (in pieces)
    seen = {form(*size) for size in test_gpu_dw_turned.SIZES}
    assert seen == {(128, True, False, False, False, False), (128, False, True, False, False, False),
                    (128, True, False, True, False, False), (128, False, True, True, False, False),
                    (256, True, False, False, False, False), (256, True, True, False, False, False),
                    (256, True, True, True, True, False), (256, True, False, True, True, True),
                    (256, False, True, True, True, True), (256, True, True, False, False, True)}
    ragged = {form(M, N, K) for M, N, K in test_gpu_dw_turned.SIZES if N % 64 and K % 64 and M % 32}
    assert seen - ragged == {(256, True, True, False, False, True)}
    assert [form(*size, 3)[:4] + form(*size, 3)[5:] for size in test_gpu_dw_turned.CLIP_SIZES] == [
        (128, True, False, True, False), (128, False, True, True, False), (256, True, False, True, True), (256, False, True, True, True)]
    M, N = test_gpu_dw_turned.SQUARE
    assert plans.dw_turns(M, N, N, 1, True, True)


def test_either_order_of_a_backward():
    """Where dX and dW, whole or in ranges, share the place of their partial sums, both orders are met: sizes against the oracle, and exact ones."""
    for sizes in ([c[:3] for c in test_gpu_dw_tiles.CASES], test_gpu_dw_turned.SIZES):
        assert {plans.dw_first(*size) for size in sizes if not plans.dw_turns(*size, alone=False)} == {False, True}


def test_outputs_over_an_input_take_copies():
    """Workgroups of dW read operands that are taken as they stand while others store dW, and after dX has been stored: X and a gradient that an
    output meets are copied."""
    M, N, K = test_gpu_dw_turned.OVER
    X, dY, dX, dW = (i << 40 for i in range(1, 5))
    x_bytes, dy_bytes, dw_bytes = M * K * 2, M * N * 2, N * K * 4
    for grad in (dY, None):
        assert plans.dw_in_place(M, N, K, X, grad, dX, dW) and plans.dw_in_place(M, N, K, X, grad, None, dW)
        for at, in_bytes in ((X, x_bytes), (dY, dy_bytes)):
            place = {"dW": lambda p: plans.dw_in_place(M, N, K, X, grad, dX, p), "dX": lambda p: plans.dw_in_place(M, N, K, X, grad, p, dW)}
            for out, out_bytes in (("dW", dw_bytes), ("dX", x_bytes)):
                # next to each other is apart
                assert place[out](at + in_bytes) and place[out](at - out_bytes)
                # (a gradient that is summed or scaled has been read by the preparation)
                assert {place[out](at + d) for d in (0, 16, in_bytes - 16, 16 - out_bytes)} == {at == dY and grad is None}


def test_loss_sizes():
    """The last workgroup to arrive finishes the losses in grids of up to so many: sizes on either side, and right at it, in either form."""
    limit, seen = plans.loss_arrivals(), {"tiled": set(), "split": set()}
    for M, N, K, rs in test_gpu_loss_arrivals.SIZES:
        form, workgroups = plans.loss_workgroups(M, N, K, len(rs))
        seen[form].add(workgroups)
    assert seen == {"tiled": {1, limit - 1, limit, limit + 1}, "split": {4, limit - 4, limit, limit + 4}}


def test_split_decode_sizes():
    forms = [plans.gemv_split(5, N, K, 4) for N, K in test_gpu_gemv_split_ring.CASES]
    assert all(p.groups >= 4 for p in forms)
    assert {(p.lines, p.depth) for p in forms} == {(n, d) for n in (1, 2) for d in (6, 4, 3)} | {(1, 0)}
    # tiles of the busiest wave against the places of a ring of six: fewer, as many, one more (one line to a slice), many more
    assert {p.blocks for p in forms if p.depth == 6 and p.lines == 1} >= {1, 5, 6, 7}
    assert {2 * p.blocks for p in forms if p.depth == 6 and p.lines == 2} >= {2, 4, 6, 8}
    # a last group of fewer than four slices, with one line and with two
    assert {p.lines for (N, K), p in zip(test_gpu_gemv_split_ring.CASES, forms) if K // 256 // p.lines % 4} == {1, 2}


def test_decode_register_sizes():
    seen = {(r, p.row_groups, p.registers) for r, p in ((r, plans.gemv(B, N, K, r)) for B, N, K, r in test_gpu_gemv_registers.CASES)}
    assert seen == {(3, 1, 128), (3, 1, 256), (3, 2, 256), (2, 2, 128), (2, 2, 256), (6, 2, 128), (6, 2, 256)}


def test_decode_list_sizes():
    plan = lambda N, K, r, B, short: plans.quad(B, N, K, r, with_list=True)
    assert all(plan(*c).waves == 0 < plans.quad(c[3], *c[:3]).waves for c in test_gpu_gemv_list.FALLBACK)
    forms = [(c, plan(*c)) for c in test_gpu_gemv_list.IN_ONE_LAUNCH]
    assert {p[0:1] + p[2:] for _, p in forms} == {(1, 3, False), (2, 2, False), (3, 5, False), (4, 4, False), (4, 4, True)}
    assert all(p.shared == (p.waves == 4 and c[3] >= 3) for c, p in forms)
    assert {p.lines for _, p in forms if p.shared} == {1, 2, 3, 4}


def test_every_wave_of_a_list_has_a_streaming_wave_or_shares():
    """Wherever the list is as long as the plane for four streaming waves, they help with it."""
    for N in (16384, 28672, 73728):
        for K in range(256, 16385, 64):
            for r in (2, 4):
                for B in (1, 2, 3, 4):
                    p = plans.quad(B, N, K, r, with_list=True)
                    if p.waves:
                        assert p.list_waves >= p.waves and p.waves + p.list_waves in (4, 8)
                        assert p.shared == (p.waves == 4 and B >= 3)
