"""GPU parity of the BF16 product on decode batches of 17 .. 64 tokens (the high-precision path
that the decode phase keeps), with and without a caller-owned workspace: the ring kernel,
whose waves take the K steps in turn, its K slabs across workgroups, and the staged kernel on the widest
weights.  Every output is
compared with the oracle's FP64 product of the BF16 inputs; where K slabs are meant, the launch rule is
asked for their number and the workspace is checked for what was written to it."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_20315_amd as mq
from paper_2605_20315_amd import _lib, workloads as wl

from _gpu_util import check_gemm_bf16, check_gemm_fp32, check_workspace_use, dev_bf16, full_of_nan, host_bits

pytestmark = pytest.mark.gpu

# (M, N, K).  K slabs with a workspace: (64, 4096, 14336), 224 K steps in 4 slabs; (48, 1000, 16384), N % 64 != 0;
# otherwise one launch: (33, 6152, 8192), ragged N; (40, 4096, 8320), 130 K steps; (64, 24640, 384), wide N,
# six K steps; (32, 16392, 1024), (17, 28672, 512): wide ragged N, two token tiles; (20, 520, 1024),
# (24, 4096, 8192): narrow N below 33 tokens; (64, 4096, 4096): short K; (64, 4098, 8192): N % 4 != 0;
# (40, 4096, 320): five K steps.
SHAPES = [(64, 4096, 14336), (33, 6152, 8192), (40, 4096, 8320), (48, 1000, 8192), (48, 1000, 16384),
          (64, 24640, 384), (32, 16392, 1024), (17, 28672, 512), (20, 520, 1024), (24, 4096, 8192),
          (64, 4096, 4096), (64, 4098, 8192), (40, 4096, 320)]
SLAB_SHAPES = {(64, 4096, 14336), (48, 1000, 16384)}


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_decode_batches_with_and_without_workspace(M, N, K):
    print(f"\n[case] bf16 decode M={M} N={N} K={K}", flush=True)
    rng = np.random.default_rng([M, N, K])
    x = wl.f32_to_bf16_bits(rng.standard_normal((M, K)).astype(np.float32))
    w = wl.f32_to_bf16_bits((rng.standard_normal((N, K)) * K ** -0.5).astype(np.float32))
    a, b = oracle.bf16_to_f64(x), oracle.bf16_to_f64(w)
    ref, na, nb = oracle.gemm_f64(a, b), oracle.row_norms(a), oracle.row_norms(b)
    xd, wd = dev_bf16(x), dev_bf16(w)
    need = mq.mq_bf16_gemm_workspace_bytes(M, N, K)
    assert need % (M * N * 4) == 0
    slabs = mq.mq_bf16_gemm_launches(M, N, K, need)[0]["slabs"]
    assert slabs >= 2 or (M, N, K) not in SLAB_SHAPES
    ws = full_of_nan(max(need, 16))
    ld = (N + 7) // 8 * 8 + 8
    for workspace in (None, ws):
        b32 = torch.full((M + 1, ld), -7.0, dtype=torch.float32, device="cuda")
        b16 = torch.full((M + 1, ld), -7.0, dtype=torch.bfloat16, device="cuda")
        y32 = mq.bf16_gemm_ws(xd, wd, workspace, mq.MQ_OUT_FP32, b32[:M, :N])
        y16 = mq.bf16_gemm_ws(xd, wd, workspace, mq.MQ_OUT_BF16, b16[:M, :N])
        again = torch.empty((M, ld), dtype=torch.bfloat16, device="cuda")
        mq.bf16_gemm_ws(xd, wd, workspace, mq.MQ_OUT_BF16, again[:, :N])
        torch.cuda.synchronize()
        check_gemm_fp32(y32.cpu().numpy(), ref, na, nb)
        check_gemm_bf16(host_bits(y16), ref, na, nb)
        assert torch.equal(y32.to(torch.bfloat16), y16)
        assert torch.equal(again[:, :N], y16)
        for buf in (b32, b16):
            assert bool((buf[M:] == -7.0).all()) and bool((buf[:, N:] == -7.0).all())
    check_workspace_use(ws, slabs, M, N)
    # the plain entry point is the workspace variant without a workspace
    y_plain = torch.empty((M, ld), dtype=torch.bfloat16, device="cuda")
    mq.bf16_gemm(xd, wd, mq.MQ_OUT_BF16, y_plain[:, :N])
    y_none = torch.empty((M, ld), dtype=torch.bfloat16, device="cuda")
    mq.bf16_gemm_ws(xd, wd, None, mq.MQ_OUT_BF16, y_none[:, :N])
    torch.cuda.synchronize()
    assert torch.equal(y_plain[:, :N], y_none[:, :N])


def test_workspace_query_and_small_workspaces():
    q = mq.mq_bf16_gemm_workspace_bytes
    assert q(64, 4096, 8192) == 16 * 64 * 4096 * 4
    assert q(64, 4096, 14336) == 16 * 64 * 4096 * 4
    assert q(48, 6144, 14336) == 10 * 48 * 6144 * 4
    assert q(16, 4096, 8192) == 0 and q(65, 4096, 8192) == 0          # other kernels serve these
    assert q(64, 4098, 8192) == 0 and q(64, 4096, 8256) == 0 and q(64, 4096, 4096) == 0
    assert q(64, 28672, 8192) == 0 and q(32, 4096, 8192) == 0      # wide N: no slabs; up to 32 tokens: none
    M, N, K = 64, 4096, 14336
    rng = np.random.default_rng(3)
    x = wl.f32_to_bf16_bits(rng.standard_normal((M, K)).astype(np.float32))
    w = wl.f32_to_bf16_bits((rng.standard_normal((N, K)) * K ** -0.5).astype(np.float32))
    a, b = oracle.bf16_to_f64(x), oracle.bf16_to_f64(w)
    ref, na, nb = oracle.gemm_f64(a, b), oracle.row_norms(a), oracle.row_norms(b)
    xd, wd = dev_bf16(x), dev_bf16(w)
    slab = M * N * 4
    most = mq.mq_bf16_gemm_launches(M, N, K, q(M, N, K))[0]["slabs"]
    assert most >= 4
    # all that can be used, an unaligned size, one slab (= none), a fraction of one
    for nbytes, slabs in ((q(M, N, K), most), (most * slab + 4, most), (slab, 1), (100, 1)):
        assert mq.mq_bf16_gemm_launches(M, N, K, nbytes)[0]["slabs"] == slabs
        ws = full_of_nan(nbytes)
        y = mq.bf16_gemm_ws(xd, wd, ws, mq.MQ_OUT_FP32)
        torch.cuda.synchronize()
        check_gemm_fp32(y.cpu().numpy(), ref, na, nb)
        check_workspace_use(ws, slabs, M, N)
    lib = _lib.load()
    y = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    args = [xd.data_ptr(), K, wd.data_ptr(), K, M, N, K, y.data_ptr(), N, mq.MQ_OUT_BF16]
    assert lib.bf16_gemm_ws(*args, ws.data_ptr() + 4, 1 << 19, 0) == 3      # MQ_ERR_ALIGN
    assert lib.bf16_gemm_ws(*args, ws.data_ptr(), -1, 0) == 2              # MQ_ERR_SHAPE
    assert lib.bf16_gemm_ws(*args, None, 1 << 20, 0) == _lib.MQ_OK         # NULL with a size: treated as none
    torch.cuda.synchronize()
    check_gemm_bf16(host_bits(y), ref, na, nb)
