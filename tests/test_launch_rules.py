"""The launch rules at shapes where both sides of a choice were timed on the GPU: the rule takes the side that was
faster.  Host only."""
import pytest

from paper_2605_20315_amd import _lib


@pytest.fixture(scope="module")
def lib():
    return _lib.load()


# rows per workgroup of the plain (0), silu_mul (1) and rmsnorm (2) quantizers: (source, rows, K, faster by 3 % or more)
@pytest.mark.parametrize("source,rows,K,want", [
    (0, 64, 4096, 4), (0, 2048, 4096, 4), (0, 3581, 4096, 4), (0, 576, 14336, 4), (0, 8189, 64, 4),
    (0, 4096, 4096, 4), (0, 3261, 5120, 16), (0, 4096, 5120, 16), (0, 8192, 4096, 16), (0, 637, 25600, 16), (0, 65536, 4096, 16), (0, 13709, 14336, 16), (0, 3421, 14336, 16), (0, 1456, 14336, 4), (0, 4672, 14336, 4),
    (1, 64, 4096, 4), (1, 1021, 14336, 4), (1, 8192, 14336, 4), (1, 16381, 4096, 4), (1, 13712, 14336, 4),
    (1, 18269, 14336, 16), (1, 10237, 25600, 16),
    (2, 64, 4096, 4), (2, 65536, 4096, 4), (2, 3000, 5120, 4), (2, 6000, 5120, 4), (2, 8192, 5120, 16), (2, 65536, 5120, 16),
    (2, 24000, 4160, 16), (2, 8192, 6144, 4), (2, 32768, 8192, 4), (2, 1000, 14336, 4), (2, 4096, 14336, 16), (2, 64, 25600, 16)])
def test_quantizer_rows_per_workgroup(lib, source, rows, K, want):
    assert lib.mq_quantize_rows(source, rows, K) == want
