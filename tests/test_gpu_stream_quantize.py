"""The row-major quantizer of tensors larger than the last-level cache reads them non-temporally: the same bytes as the other
quantizer and the conversion between the two orders give, on either side of the line (256 MiB of BF16) and with strided rows."""
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
