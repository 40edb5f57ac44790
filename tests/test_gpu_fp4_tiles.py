"""GPU parity of the NVFP4 product at one problem per workgroup tile of its two kernels and of each kind of
launch in two parts (rows or columns of Y), with ragged M and N, K of one step up to counts that the
waves and register sets do not divide, in either byte order and with both output types.  Every output is
compared with the oracle's FP64 product of the dequantized operands; nothing outside [M, N] may be
written."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_20315_amd as mq

from _gpu_util import check_gemm_bf16, check_gemm_fp32, dev_scalar, dev_u8, host_bits, to_ktile

pytestmark = pytest.mark.gpu

KTILE, LINEAR = mq.MQ_LAYOUT_KTILE, mq.MQ_LAYOUT_LINEAR
# (byte order, M, N, K, launches on 256 compute units: kernel, tile (tokens x rows of W) x waves, and the direction of
# a launch in two parts); each byte order has the tiles that it can select
CASES = [
    (KTILE, 1, 8, 64, "small 32x32x8"),
    (KTILE, 1, 8, 192, "small 32x32x8"),
    (KTILE, 65, 4397, 128, "small 32x64x4"),
    (KTILE, 33, 4099, 704, "small 32x64x4"),
    (KTILE, 16, 520, 512, "small 32x32x8"),
    (KTILE, 33, 4277, 192, "small 32x64x4"),
    (KTILE, 81, 5117, 12800, "small 32x64x8"),
    (KTILE, 65, 5492, 192, "small 64x32x4"),
    (KTILE, 2746, 129, 832, "small 64x32x8"),
    (KTILE, 161, 5536, 64, "small 64x64x1"),
    (KTILE, 250, 1001, 192, "small 32x32x8"),
    (KTILE, 65, 5454, 448, "small 64x64x4"),
    (KTILE, 101, 5117, 6400, "small 64x64x8"),
    (KTILE, 172, 5586, 832, "small 64x128x4"),
    (KTILE, 35, 28670, 4096, "small 64x128x8"),
    (KTILE, 3599, 261, 832, "small 128x64x4"),
    (KTILE, 840, 1194, 704, "small 128x64x8"),
    (KTILE, 328, 5978, 3008, "direct 128x128x4"),
    (KTILE, 916, 7684, 576, "direct 256x128x4"),
    (KTILE, 2182, 6084, 192, "direct 256x256x4"),
    (KTILE, 2587, 6169, 64, "direct 256x256x4; small 32x32x8 rows"),
    (KTILE, 3139, 1293, 1600, "direct 128x128x4; small 32x32x8 columns"),
    (KTILE, 1171, 6882, 704, "direct 256x128x4; small 32x64x4 columns"),
    (KTILE, 2646, 5929, 256, "direct 256x256x4; small 32x32x8 columns"),
    (KTILE, 771, 5127, 1600, "direct 128x128x4; small 32x32x8 rows"),
    (KTILE, 1027, 8058, 704, "direct 256x128x4; small 32x32x8 rows"),
    (KTILE, 2071, 8187, 192, "direct 256x256x4; small 32x32x8 rows"),
    (LINEAR, 1, 8, 64, "small 32x32x8"),
    (LINEAR, 33, 4195, 64, "small 32x64x4"),
    (LINEAR, 33, 4099, 704, "small 64x32x4"),
    (LINEAR, 1, 8, 256, "small 64x32x4"),
    (LINEAR, 1, 8, 192, "small 64x32x8"),
    (LINEAR, 130, 6663, 64, "small 64x64x1"),
    (LINEAR, 65, 5788, 576, "small 64x64x4"),
    (LINEAR, 277, 5485, 448, "small 64x128x4"),
    (LINEAR, 129, 6793, 192, "small 128x64x4"),
    (LINEAR, 330, 5512, 576, "direct 128x128x4"),
    (LINEAR, 834, 7021, 256, "direct 256x128x4"),
    (LINEAR, 1223, 7363, 192, "direct 256x256x4"),
    (LINEAR, 21, 18463, 2752, "small 64x128x4"),
    (LINEAR, 2346, 1666, 1600, "direct 128x128x4; small 32x32x8 columns"),
    (LINEAR, 4041, 2075, 832, "direct 256x128x4; small 64x32x4 columns"),
    (LINEAR, 3857, 4879, 448, "direct 256x256x4; direct 128x128x4 columns"),
    (LINEAR, 2731, 6005, 192, "direct 256x256x4; small 64x32x4 columns"),
    (LINEAR, 521, 6758, 1600, "direct 128x128x4; small 32x32x8 rows"),
    (LINEAR, 1074, 7263, 832, "direct 256x128x4; small 64x32x4 rows"),
    (LINEAR, 3107, 5971, 448, "direct 256x256x4; direct 128x128x4 rows"),
    (LINEAR, 2329, 6674, 192, "direct 256x256x4; small 64x32x4 rows"),
    (KTILE, 637, 4101, 576, "small 64x64x1"),
    (KTILE, 35, 9001, 320, "small 64x32x4"),
    (LINEAR, 261, 4093, 320, "small 128x64x4"),
    (LINEAR, 452, 10285, 320, "direct 256x128x4"),
    (LINEAR, 329, 10941, 448, "direct 256x128x4"),
    (LINEAR, 258, 9797, 448, "direct 128x128x4"),
    (LINEAR, 130, 10917, 1280, "direct 128x128x4"),
    (KTILE, 578, 9937, 1280, "direct 256x128x4"),
]


def _launches(M, N, K, layout):
    parts = mq.mq_gemm_launches(M, N, K, layout)
    tag = "; ".join(f"{p['kernel'][4:]} {p['tile'][0]}x{p['tile'][1]}x{p['waves']}" for p in parts)
    return tag + ("" if len(parts) == 1 else " rows" if parts[0]["cols"] == N else " columns")


@pytest.mark.parametrize("layout,M,N,K,launches", CASES)
def test_fp4_tile_shapes_against_oracle(layout, M, N, K, launches):
    assert _launches(M, N, K, layout) == launches
    print(f"\n[case] fp4 tiles M={M} N={N} K={K} layout={layout}", flush=True)
    rng = np.random.default_rng([M, N, K])
    ac = rng.integers(0, 256, size=(M, K // 2)).astype(np.uint8)
    asc = rng.integers(0x28, 0x48, size=(M, K // 16)).astype(np.uint8)
    bc = rng.integers(0, 256, size=(N, K // 2)).astype(np.uint8)
    bsc = rng.integers(0x28, 0x48, size=(N, K // 16)).astype(np.uint8)
    aa, ba = np.float32(0.75), np.float32(1.5)
    a, b = oracle.dequantize(ac, asc, aa), oracle.dequantize(bc, bsc, ba)
    ref, na, nb = oracle.gemm_f64(a, b), oracle.row_norms(a), oracle.row_norms(b)
    arrs = (to_ktile(ac, asc) + to_ktile(bc, bsc)) if layout == mq.MQ_LAYOUT_KTILE else (ac, asc, bc, bsc)
    d = [dev_u8(t) for t in arrs]
    a_al, b_al = dev_scalar(aa), dev_scalar(ba)
    ld = (N + 7) // 8 * 8 + 8
    b32 = torch.full((M + 1, ld), -7.0, dtype=torch.float32, device="cuda")
    b16 = torch.full((M + 1, ld), -7.0, dtype=torch.bfloat16, device="cuda")
    y32 = mq.nvfp4_gemm(d[0], d[1], a_al, d[2], d[3], b_al, mq.MQ_OUT_FP32, b32[:M, :N], layout)
    y16 = mq.nvfp4_gemm(d[0], d[1], a_al, d[2], d[3], b_al, mq.MQ_OUT_BF16, b16[:M, :N], layout)
    torch.cuda.synchronize()
    check_gemm_fp32(y32.cpu().numpy(), ref, na, nb)
    check_gemm_bf16(host_bits(y16), ref, na, nb)
    assert torch.equal(y32.to(torch.bfloat16), y16)
    for buf in (b32, b16):
        assert bool((buf[M:] == -7.0).all()) and bool((buf[:, N:] == -7.0).all())
