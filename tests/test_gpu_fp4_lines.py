"""GPU parity of the small NVFP4 tiles that read row-major operands by whole lines (four K steps of a row): every tile that
does, K slabs included, over counts of lines that leave the waves none, one, two or three of them, with ragged M and N, both
output types, and scales that begin at a multiple of four bytes only.  Against the oracle's FP64 product of the dequantized
operands; nothing outside [M, N] may be written."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_20315_amd as mq

from _gpu_util import check_gemm_bf16, check_gemm_fp32, dev_scalar, dev_u8, host_bits

pytestmark = pytest.mark.gpu

LINEAR = mq.MQ_LAYOUT_LINEAR
WS = 64 << 20
# (M, N, lines of K (256 elements each), bytes of workspace, launch on 256 compute units)
CASES = [
    (1, 8, (8, 9), 0, "32x32x8"),
    (33, 72, (8, 9, 15, 16, 17, 23, 25, 33), 0, "32x32x8"),
    (1, 9201, (9,), 0, "32x64x8"),
    (65, 5001, (8, 9, 10), 0, "32x64x4"),
    (33, 4097, (8, 9), 0, "64x32x8"),
    (33, 4097, (11, 13, 16), 0, "64x32x4"),
    (97, 4097, (8,), 0, "64x64x8"),
    (65, 6001, (9,), 0, "64x64x8"),
    (97, 4097, (20,), 0, "64x64x4"),
    (161, 3001, (17,), 0, "64x64x4"),
    (65, 6273, (20,), 0, "64x64x4"),   # the last tiles hold one row and one column
    (589, 3669, (8,), 0, "64x64x4"),   # 580 tiles: the lanes past the end read the rows in front of the last tiles
    (1, 8, (32, 33, 47), WS, "32x32x8 in slabs"),
    (65, 1000, (47,), WS, "32x64x8 in slabs"),
    (65, 1000, (32,), WS, "64x32x8 in slabs"),
    (129, 1000, (47,), WS, "64x64x8 in slabs"),
    (193, 2000, (56,), WS, "64x64x4 in slabs"),
]


def _launch(M, N, K, ws):
    (p,) = mq.mq_gemm_launches(M, N, K, LINEAR, ws)
    assert p["kernel"] == "fp4_small"
    return f"{p['tile'][0]}x{p['tile'][1]}x{p['waves']}" + (" in slabs" if p["slabs"] > 1 else "")


@pytest.mark.parametrize("M,N,lines,ws,launch", CASES)
def test_rows_read_by_lines(M, N, lines, ws, launch):
    rng = np.random.default_rng([M, N, ws])
    one = np.float32(1.0)
    workspace = torch.empty(ws, dtype=torch.uint8, device="cuda") if ws else None
    for n in lines:
        K = 256 * n
        assert _launch(M, N, K, ws) == launch
        print(f"[case] fp4 lines M={M} N={N} K={K} {launch}", flush=True)
        ac, bc = (rng.integers(0, 256, size=(r, K // 2)).astype(np.uint8) for r in (M, N))
        asc, bsc = (rng.integers(0x28, 0x48, size=(r, K // 16)).astype(np.uint8) for r in (M, N))
        a, b = oracle.dequantize(ac, asc, one), oracle.dequantize(bc, bsc, one)
        ref, na, nb = oracle.gemm_f64(a, b), oracle.row_norms(a), oracle.row_norms(b)
        d_as, d_bs = (dev_u8(np.concatenate([np.zeros(4, np.uint8), s.ravel()]))[4:].view(s.shape) for s in (asc, bsc))
        d_ac, d_bc, al = dev_u8(ac), dev_u8(bc), dev_scalar(1.0)
        ld = (N + 7) // 8 * 8 + 8
        outs = {}
        for out, dtype in ((mq.MQ_OUT_FP32, torch.float32), (mq.MQ_OUT_BF16, torch.bfloat16)):
            buf = torch.full((M + 1, ld), -7.0, dtype=dtype, device="cuda")
            outs[out] = mq.nvfp4_gemm_ws(d_ac, d_as, al, d_bc, d_bs, al, workspace, out, buf[:M, :N], LINEAR)
            torch.cuda.synchronize()
            assert bool((buf[M:] == -7.0).all()) and bool((buf[:, N:] == -7.0).all())
        check_gemm_fp32(outs[mq.MQ_OUT_FP32].cpu().numpy(), ref, na, nb)
        check_gemm_bf16(host_bits(outs[mq.MQ_OUT_BF16]), ref, na, nb)
        assert torch.equal(outs[mq.MQ_OUT_FP32].to(torch.bfloat16), outs[mq.MQ_OUT_BF16])
