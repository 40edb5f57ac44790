"""GPU parity of the K-step-major quantizers on both sides of the launcher's choice of rows per workgroup
(four, or sixteen for large tensors) and of rows kept in registers by the RMSNorm quantizer, and of the
layout conversion over ragged tiles.  Codes and scale bytes are compared bit for bit with the oracle
quantizer applied to the BF16 tensor (for the fused producers: the one that the kernel reports)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_20315_amd as mq
from paper_2605_20315_amd import _lib, workloads as wl

from _gpu_util import dev_bf16, dev_scalar, dev_u8, host_bits, to_ktile

pytestmark = pytest.mark.gpu


def _same(c, s, bits, alpha):
    ce, se = to_ktile(*oracle.quantize(bits, alpha))
    assert np.array_equal(s.cpu().numpy(), se) and np.array_equal(c.cpu().numpy(), ce)


# four rows per workgroup up to 960 (rows % 4 == 0: 1100) workgroups of sixteen, then sixteen; 1 and 17 K steps, ragged rows
@pytest.mark.parametrize("rows,K,per", [(3, 64, 4), (18, 1088, 4), (15343, 64, 4), (15347, 64, 16), (7660, 1088, 4), (7670, 1088, 16), (8784, 1088, 4), (8800, 1088, 16),
                                        (65543, 64, 16), (32770, 1088, 16)])
def test_quantize_rows_per_workgroup(rows, K, per):
    assert _lib.load().mq_quantize_rows(0, rows, K) == per
    rng = np.random.default_rng([rows, K])
    bits = wl.f32_to_bf16_bits(rng.standard_normal((rows, K), dtype=np.float32))
    c, s = mq.nvfp4_quantize(dev_bf16(bits), dev_scalar(0.002), layout=mq.MQ_LAYOUT_KTILE)
    torch.cuda.synchronize()
    _same(c, s, bits, np.float32(0.002))


# sixteen rows from 16384 workgroups, from 10240 where rows % 4 != 0
@pytest.mark.parametrize("rows,K,per", [(5, 1088, 4), (163823, 64, 4), (163825, 64, 16), (262124, 64, 4), (262136, 64, 16)])
def test_silu_mul_rows_per_workgroup(rows, K, per):
    assert _lib.load().mq_quantize_rows(1, rows, K) == per
    gu = torch.randn((rows, 2 * K), device="cuda", generator=torch.Generator(device="cuda").manual_seed(rows)).to(torch.bfloat16)
    c, s, p = mq.nvfp4_quantize_silu_mul(gu, dev_scalar(0.002), layout=mq.MQ_LAYOUT_KTILE, return_bf16=True)
    ref = oracle.bf16_round(oracle.silu_mul_f64(host_bits(gu)))
    bits = host_bits(p)
    assert float((bits == ref).mean()) >= 0.999
    _same(c, s, bits, np.float32(0.002))


# four rows with the row in 4, 8 or 16 chunks of registers, then sixteen with x read twice
@pytest.mark.parametrize("rows,K", [(3, 4096), (6, 4160), (33, 8192), (5, 8256), (1021, 16384), (2, 16448), (1027, 8256), (6145, 4160)])
@pytest.mark.parametrize("layout", [mq.MQ_LAYOUT_KTILE, mq.MQ_LAYOUT_LINEAR])
def test_rmsnorm_rows_per_workgroup(rows, K, layout):
    g = torch.Generator(device="cuda").manual_seed(rows * K)
    x = torch.randn((rows, K), device="cuda", generator=g).to(torch.bfloat16)
    w = (1.0 + 0.1 * torch.randn(K, device="cuda", generator=g)).to(torch.bfloat16)
    c, s, y = mq.nvfp4_quantize_rmsnorm(x, w, 1e-6, dev_scalar(0.002), layout=layout, return_bf16=True)
    ref = oracle.bf16_round(oracle.rmsnorm_f64(host_bits(x), host_bits(w), 1e-6))
    bits = host_bits(y)
    assert float((bits == ref).mean()) >= 0.9999 or int((bits != ref).sum()) <= 1
    ce, se = oracle.quantize(bits, np.float32(0.002))
    if layout == mq.MQ_LAYOUT_KTILE:
        ce, se = to_ktile(ce, se)
    assert np.array_equal(s.cpu().numpy(), se) and np.array_equal(c.cpu().numpy(), ce)


# one thread per unit of (row, K step) below 2^17 units (3 * 2^16 to the K-step-major order) or four K steps, else tiles of 32 rows x 16 K steps
@pytest.mark.parametrize("rows,K", [(31, 960), (33, 1088), (64, 2048), (1, 8256), (1, 64), (140001, 64), (70001, 192), (131071, 64),
                                    (32767, 256), (32769, 256), (49151, 256), (49153, 256), (7711, 1088), (1025, 8192), (33, 256064)])
def test_relayout_ragged_tiles(rows, K):
    rng = np.random.default_rng([rows, K])
    c = rng.integers(0, 256, size=(rows, K // 2)).astype(np.uint8)
    s = rng.integers(0, 127, size=(rows, K // 16)).astype(np.uint8)
    ck, sk = mq.nvfp4_relayout(dev_u8(c), dev_u8(s), mq.MQ_LAYOUT_LINEAR, mq.MQ_LAYOUT_KTILE)
    cl, sl = mq.nvfp4_relayout(ck, sk, mq.MQ_LAYOUT_KTILE, mq.MQ_LAYOUT_LINEAR)
    torch.cuda.synchronize()
    ce, se = to_ktile(c, s)
    assert np.array_equal(ck.cpu().numpy(), ce) and np.array_equal(sk.cpu().numpy(), se)
    assert np.array_equal(cl.cpu().numpy(), c) and np.array_equal(sl.cpu().numpy(), s)


def test_relayout_of_more_k_steps_than_one_launch_holds():
    """One row of 2^24 tiles of 16 K steps (8.6 GB of codes), one tile more than a launch of 2^24 - 1 workgroups
    holds.  With a single row the two orders are the same bytes."""
    K = 1024 << 24
    if torch.cuda.mem_get_info()[0] < 64 << 30:
        pytest.skip("needs 64 GB of device memory")
    c = torch.arange(K // 16, dtype=torch.int64, device="cuda").mul_(0x9E3779B97F4A7C15 - (1 << 64)).view(torch.uint8).view(1, K // 2)
    s = torch.arange(K // 64, dtype=torch.int32, device="cuda").view(torch.uint8).view(1, K // 16)
    for a, b in ((mq.MQ_LAYOUT_LINEAR, mq.MQ_LAYOUT_KTILE), (mq.MQ_LAYOUT_KTILE, mq.MQ_LAYOUT_LINEAR)):
        oc, os_ = mq.nvfp4_relayout(c, s, a, b)
        assert torch.equal(oc.view(torch.int64), c.view(torch.int64))
        assert torch.equal(os_.view(torch.int32), s.view(torch.int32))
        del oc, os_
    del c, s
    torch.cuda.empty_cache()
