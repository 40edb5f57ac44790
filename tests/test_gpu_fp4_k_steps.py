"""GPU parity of the small NVFP4 tiles over the number of K steps: a wave's part of K is cut into groups of two to four K
steps whose last one stops at the wave's last step, and waves beyond the end of K have none.  Against the oracle's FP64
product of the dequantized operands."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_20315_amd as mq

from _gpu_util import check_gemm_fp32, dev_scalar, dev_u8, to_ktile

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", [mq.MQ_LAYOUT_KTILE, mq.MQ_LAYOUT_LINEAR])
@pytest.mark.parametrize("M,N", [(33, 72), (65, 136), (97, 5000), (300, 3072)])
def test_every_count_of_k_steps(layout, M, N):
    counts = list(range(1, 42)) + [63, 64, 65, 95, 97] if N < 1000 else [1, 2, 3, 5, 7, 9, 10, 11, 13, 19, 33]
    kmax = 64 * max(counts)
    rng = np.random.default_rng([M, N, layout])
    ac, bc = (rng.integers(0, 256, size=(r, kmax // 2)).astype(np.uint8) for r in (M, N))
    asc, bsc = (rng.integers(0x28, 0x48, size=(r, kmax // 16)).astype(np.uint8) for r in (M, N))
    one, al = np.float32(1.0), dev_scalar(1.0)
    a, b = oracle.dequantize(ac, asc, one), oracle.dequantize(bc, bsc, one)
    seen = set()
    for kt in counts:
        K = 64 * kt
        print(f"[case] fp4 K steps M={M} N={N} K={K} layout={layout}", flush=True)
        seen.update(p["kernel"] for p in mq.mq_gemm_launches(M, N, K, layout))
        ops = [np.ascontiguousarray(t[:, :w]) for t, w in ((ac, K // 2), (asc, K // 16), (bc, K // 2), (bsc, K // 16))]
        if layout == mq.MQ_LAYOUT_KTILE:
            ops = to_ktile(*ops[:2]) + to_ktile(*ops[2:])
        d = [dev_u8(t) for t in ops]
        y = mq.nvfp4_gemm(d[0], d[1], al, d[2], d[3], al, mq.MQ_OUT_FP32, None, layout)
        ak, bk = np.ascontiguousarray(a[:, :K]), np.ascontiguousarray(b[:, :K])
        check_gemm_fp32(y.cpu().numpy(), oracle.gemm_f64(ak, bk), oracle.row_norms(ak), oracle.row_norms(bk))
    assert seen == {"fp4_small"}
