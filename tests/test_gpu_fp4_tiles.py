"""GPU parity of the NVFP4 product at one problem per workgroup tile of its two kernels and of each kind of
launch in two parts (rows or columns of Y), with ragged M and N, K of one step up to counts that the
waves and register sets do not divide, both byte orders and both output types.  Every output is
compared with the oracle's FP64 product of the dequantized operands; nothing outside [M, N] may be
written."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_20315_amd as mq

from _gpu_util import check_gemm_bf16, check_gemm_fp32, dev_scalar, dev_u8, host_bits, to_ktile

pytestmark = pytest.mark.gpu

# tile (tokens x rows of W) x waves on 256 compute units: 64x32x4, 32x64x4 (K of 2 and 11 steps), 32x32x8 (8 steps),
# 64x32x8, 32x64x8, 64x64x8, 64x64x4, 64x128x4, 128x64x4, 64x128x8, 128x64x8, 128x128, 256x128, 256x256; then rows
# split at 2560 (256x256 + 64x32) and 1536 (128x128 + 32x32), columns at 7168 (256x256 + 64x32) and
# 3200 (256x128 + 32x32)
SHAPES = [(1, 8, 64), (65, 4397, 128), (33, 4099, 704), (16, 520, 512), (33, 4233, 3136), (65, 4364, 4352),
          (69, 5451, 4224), (67, 5480, 320), (269, 5655, 192), (194, 7081, 320), (134, 6619, 3008), (321, 5400, 3136),
          (450, 6254, 256), (641, 7039, 192), (1031, 6537, 192), (2587, 6169, 64), (1546, 2644, 832), (2102, 7170, 64),
          (2537, 3272, 576)]


@pytest.mark.parametrize("layout", [mq.MQ_LAYOUT_KTILE, mq.MQ_LAYOUT_LINEAR])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_fp4_tile_shapes_against_oracle(M, N, K, layout):
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
