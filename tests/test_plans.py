"""Rules on sizes (no GPU): what the launches that follow from them rely on."""
import pytest

from tests import plans

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
