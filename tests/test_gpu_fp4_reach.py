"""Small tiles whose part of K spans more than 2 GiB: the loads' base moves up within the K loop.  Many rows of W for few
tokens, and many tokens for few rows of W; sampled rows of the large operand against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_20315_amd as mq

from _gpu_util import check_gemm_bf16, host_bits

pytestmark = pytest.mark.gpu

KTILE = mq.MQ_LAYOUT_KTILE


def _operand(rows, K, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    codes = torch.randint(0, 256, (rows, K // 2), dtype=torch.uint8, device="cuda", generator=g)
    scales = torch.randint(0x28, 0x48, (rows, K // 16), dtype=torch.uint8, device="cuda", generator=g)
    return codes, scales


def _values(codes, scales, at):
    """The given rows of a K-step-major operand, dequantized by the oracle."""
    rows, K = codes.shape[0], codes.shape[1] * 2
    idx = torch.from_numpy(at).cuda()
    c = codes.view(K // 64, rows, 32)[:, idx].permute(1, 0, 2).reshape(len(at), K // 2)
    s = scales.view(K // 64, rows, 4)[:, idx].permute(1, 0, 2).reshape(len(at), K // 16)
    return oracle.dequantize(np.ascontiguousarray(c.cpu().numpy()), np.ascontiguousarray(s.cpu().numpy()), 1.0)


# eight waves with 128 K steps each (2.5 GB of codes between the first and the last), four waves with 129 or 128 of them (2.4)
@pytest.mark.parametrize("M,N,K", [(5, 600016, 65536), (600011, 64, 32832)])
def test_part_of_k_beyond_2_gib(M, N, K):
    print(f"\n[case] part of K beyond 2 GiB M={M} N={N} K={K}", flush=True)
    (p,) = mq.mq_gemm_launches(M, N, K, KTILE)
    assert p["kernel"] == "fp4_small" and -(-K // 64 // p["waves"]) * max(M, N) * 32 > 1 << 31
    a, b = _operand(M, K, 1), _operand(N, K, 2)
    one = torch.ones(1, device="cuda")
    y = mq.nvfp4_gemm(*a, one, *b, one, layout=KTILE)
    torch.cuda.synchronize()
    at = lambda n: np.arange(n) if n < 100 else np.unique(np.r_[0:3, 31:34, n // 3, n // 2:n // 2 + 3, n - 45, n - 12:n])
    rows, cols = at(M), at(N)
    va, vb = _values(*a, rows), _values(*b, cols)
    got = y[torch.from_numpy(rows).cuda()][:, torch.from_numpy(cols).cuda()]
    check_gemm_bf16(host_bits(got), oracle.gemm_f64(va, vb), oracle.row_norms(va), oracle.row_norms(vb))
    del a, b, y
    torch.cuda.empty_cache()
