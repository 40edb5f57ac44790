"""The row-major quantizer of tensors larger than the last-level cache reads them non-temporally: the same bytes as the other
quantizer and the conversion between the two orders give, on either side of the line (256 MiB of BF16) and with strided rows.  The
conversion does so from 5.6 MB on: the documented permutation on either side of that line, in both directions."""
import pytest
import torch

import paper_2605_20315_amd as mq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,K,pad", [(32768, 4096, 0), (32769, 4096, 0), (8193, 16384, 64), (131073, 1024, 8)])
def test_row_major_quantizer_on_both_sides_of_the_line(rows, K, pad):
    print(f"\n[case] row-major quantizer {rows} x {K} pad {pad}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(rows + K)
    x = torch.randn((rows, K + pad), device="cuda", generator=g).to(torch.bfloat16)[:, :K]
    x[::1001] *= 100.0
    alpha = mq.nvfp4_global_scale(x)
    codes, scales = mq.nvfp4_quantize(x, alpha, layout=mq.MQ_LAYOUT_LINEAR)
    kcodes, kscales = mq.nvfp4_quantize(x, alpha, layout=mq.MQ_LAYOUT_KTILE)
    back_codes, back_scales = mq.nvfp4_relayout(kcodes, kscales, mq.MQ_LAYOUT_KTILE, mq.MQ_LAYOUT_LINEAR)
    torch.cuda.synchronize()
    assert torch.equal(codes.view(-1), back_codes.view(-1)) and torch.equal(scales.view(-1), back_scales.view(-1))


@pytest.mark.parametrize("rows,K", [(2048, 4096), (2559, 4096), (2730, 3840), (4096, 2560), (2561, 4096), (3071, 4096), (3073, 4160)])
def test_conversion_on_both_sides_of_its_line(rows, K):
    print(f"\n[case] conversion {rows} x {K}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(rows + K)
    codes = torch.randint(0, 256, (rows, K // 2), device="cuda", generator=g, dtype=torch.uint8)
    scales = torch.randint(0, 256, (rows, K // 16), device="cuda", generator=g, dtype=torch.uint8)
    want_c = codes.view(rows, K // 64, 32).permute(1, 0, 2).reshape(-1)
    want_s = scales.view(rows, K // 64, 4).permute(1, 0, 2).reshape(-1)
    kcodes, kscales = mq.nvfp4_relayout(codes, scales, mq.MQ_LAYOUT_LINEAR, mq.MQ_LAYOUT_KTILE)
    back_c, back_s = mq.nvfp4_relayout(kcodes, kscales, mq.MQ_LAYOUT_KTILE, mq.MQ_LAYOUT_LINEAR)
    torch.cuda.synchronize()
    assert torch.equal(kcodes.view(-1), want_c) and torch.equal(kscales.view(-1), want_s)
    assert torch.equal(back_c, codes) and torch.equal(back_s, scales)
