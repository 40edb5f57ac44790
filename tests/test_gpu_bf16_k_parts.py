"""GPU parity of the BF16 product where K is cut into slabs across workgroups in the staged tiles, where workgroups take
the K steps of a long K in orders of their own, in the decode tile of 112 rows of W, and where a W that one row of tiles reads is
larger than 96 MB (read past the last-level cache): the last slab shorter than the others, groups of four steps with
none to three left over, ragged M and N, strided operands and output, a workspace that holds fewer slabs than the rule would
take.  Every output is compared with the oracle's FP64 product; nothing outside [M, N] and the slabs' sums may be written."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_20315_amd as mq
from paper_2605_20315_amd import workloads as wl

from _gpu_util import check_gemm_bf16, check_gemm_fp32, check_workspace_use, dev_bf16, full_of_nan, host_bits

pytestmark = pytest.mark.gpu

# (M, N, K, kernel and tile on 256 compute units); slabs where a workspace is passed
SLABS = [(70, 4100, 12480, "bf16_stage", (96, 128)), (82, 700, 8576, "bf16_stage", (96, 64)), (69, 80, 15168, "bf16_stage", (128, 64)), (131, 808, 11776, "bf16_stage", (96, 128)),
         (294, 524, 13376, "bf16_stage", (128, 128)), (129, 2360, 13760, "bf16_stage", (160, 128))]
ORDERS = [(969, 6667, 512, "bf16_d2l", (256, 192)), (1027, 7244, 4160, "bf16_d2l", (256, 192)), (1539, 6957, 4224, "bf16_d2l", (256, 256)),
          (257, 1030, 4096, None, None), (257, 1030, 4288, None, None)]
WIDE = [(44, 28077, 1088, "bf16_ring", (48, 112)), (33, 28077, 1152, "bf16_ring", (48, 112)), (100, 12305, 4160, "bf16_stage", None)]


def _operands(M, N, K):
    print(f"\n[case] bf16 parts of K M={M} N={N} K={K}", flush=True)
    rng = np.random.default_rng([M, N, K])
    x = wl.f32_to_bf16_bits(rng.standard_normal((M, K + 8)).astype(np.float32))
    w = wl.f32_to_bf16_bits((rng.standard_normal((N, K + 24)) * K ** -0.5).astype(np.float32))
    a, b = oracle.bf16_to_f64(np.ascontiguousarray(x[:, :K])), oracle.bf16_to_f64(np.ascontiguousarray(w[:, :K]))
    return dev_bf16(x)[:, :K], dev_bf16(w)[:, :K], (oracle.gemm_f64(a, b), oracle.row_norms(a), oracle.row_norms(b))


def _check(xd, wd, ws, want):
    M, N = xd.shape[0], wd.shape[0]
    ld = (N + 7) // 8 * 8 + 8
    b32 = torch.full((M + 1, ld), -7.0, dtype=torch.float32, device="cuda")
    b16 = torch.full((M + 1, ld), -7.0, dtype=torch.bfloat16, device="cuda")
    y32 = mq.bf16_gemm_ws(xd, wd, ws, mq.MQ_OUT_FP32, b32[:M, :N])
    y16 = mq.bf16_gemm_ws(xd, wd, ws, mq.MQ_OUT_BF16, b16[:M, :N])
    torch.cuda.synchronize()
    check_gemm_fp32(y32.cpu().numpy(), *want)
    check_gemm_bf16(host_bits(y16), *want)
    assert torch.equal(y32.to(torch.bfloat16), y16)
    for buf in (b32, b16):
        assert bool((buf[M:] == -7.0).all()) and bool((buf[:, N:] == -7.0).all())


@pytest.mark.parametrize("M,N,K,kernel,tile", SLABS)
def test_slabs_of_the_staged_tiles(M, N, K, kernel, tile):
    need = mq.mq_bf16_gemm_workspace_bytes(M, N, K)
    assert 2 * M * N * 4 <= need <= 16 << 20
    xd, wd, want = _operands(M, N, K)
    for nbytes in (need, 2 * M * N * 4, M * N * 4):  # all, two slabs at most, none
        plan = mq.mq_bf16_gemm_launches(M, N, K, nbytes)[0]
        assert plan["slabs"] * M * N * 4 <= max(nbytes, M * N * 4)
        if nbytes == need:
            assert plan["slabs"] > 2 and (plan["kernel"], plan["tile"]) == (kernel, tile)
            steps = K // 64
            assert steps % -(-steps // plan["slabs"]) != 0, "the last slab is meant to be shorter"
        ws = full_of_nan(nbytes)
        _check(xd, wd, ws, want)
        check_workspace_use(ws, plan["slabs"], M, N)


@pytest.mark.parametrize("M,N,K,kernel,tile", ORDERS + WIDE)
def test_orders_of_the_k_steps_and_wide_w(M, N, K, kernel, tile):
    plan = mq.mq_bf16_gemm_launches(M, N, K, 0)[0]
    assert kernel in (None, plan["kernel"]) and tile in (None, plan["tile"])
    xd, wd, want = _operands(M, N, K)
    _check(xd, wd, None, want)
