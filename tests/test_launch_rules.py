"""The launch rules at shapes where both sides of a choice were timed on the GPU: the rule takes the side that was
faster.  Host only."""
import pytest

import paper_2605_20315_amd as mq
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


# BF16 product, whatever the output type: (M, N, K, kernel and tile that was within 2 % of the fastest, where what ran
# there before or the next best choice was 4 % slower or more)
@pytest.mark.parametrize("M,N,K,kernel,tile", [
    (1, 4096, 512, "bf16_short", (16, 16)), (1, 4096, 14336, "bf16_ring", (16, 16)), (3, 5120, 25600, "bf16_ring", (16, 32)),
    (8192, 6400, 5120, "bf16_d2l", (256, 256)), (4096, 12800, 5120, "bf16_d2l", (256, 256)),
    (2048, 28672, 4096, "bf16_d2l", (256, 256)), (2048, 4096, 512, "bf16_d2l", (256, 128)),
    (8192, 5120, 640, "bf16_d2l", (256, 256)), (2048, 4096, 4096, "bf16_stage", (256, 128))])
def test_bf16_tile(M, N, K, kernel, tile):
    p = mq.mq_bf16_gemm_launches(M, N, K, 16 << 20)
    assert len(p) == 1 and (p[0]["kernel"], p[0]["tile"]) == (kernel, tile)


# NVFP4 product, K-step-major: (M, N, K, tiles of the launches) where what ran before was 4 % slower or more
@pytest.mark.parametrize("M,N,K,tiles", [
    (333, 28672, 4096, [(256, 128), (128, 128)]), (512, 28672, 4096, [(256, 256)]), (256, 8192, 128, [(64, 64)]),
    (640, 4096, 512, [(64, 64)]), (640, 4096, 256, [(64, 64)]), (6144, 2048, 128, [(256, 256)]), (2048, 5120, 1280, [(256, 256)]), (64, 4096, 4096, [(32, 32)])])
def test_fp4_tiles(M, N, K, tiles):
    assert [p["tile"] for p in mq.mq_gemm_launches(M, N, K, mq.MQ_LAYOUT_KTILE, 4 << 20)] == tiles


# A wave of the small tiles reaches 2 GiB from one base and moves it up for more, four K steps at least: (M, N, K, small tiles)
@pytest.mark.parametrize("M,N,K,small", [
    (16, 1048576, 65536, True), (16, 600000, 65536, True), (2500000, 16, 28672, True), (600000, 64, 28672, True),
    (16, (2**31 - 1) // 96, 4096, True), (16, (2**31 - 1) // 96 + 1, 4096, False), (16, 40000000, 4096, False)])
def test_fp4_small_tiles_reach(M, N, K, small):
    kernels = {p["kernel"] for p in mq.mq_gemm_launches(M, N, K, mq.MQ_LAYOUT_KTILE)}
    assert kernels == ({"fp4_small"} if small else {"fp4_direct"})
