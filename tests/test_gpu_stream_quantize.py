"""The row-major quantizer of tensors larger than the last-level cache reads them non-temporally: the same bytes as the other
quantizer and the conversion between the two orders give, on either side of the line (256 MiB of BF16) and with strided rows.  The
conversion writes them so where rows or K steps are whole cache lines, and reads them so where both are, from 19.1 MB on: the documented
permutation on either side of those lines, in both directions, and into buffers that start within a line."""
import pytest
import torch

import paper_2605_20315_amd as mq
from paper_2605_20315_amd import _lib

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


@pytest.mark.parametrize("rows,K,offset", [
    (2048, 4096, 0), (3073, 4096, 0), (3074, 4160, 0), (3076, 4160, 0), (3076, 4352, 0), (3076, 4352, 16), (3076, 4352, 64),
    (8700, 4096, 0), (8704, 4096, 0), (8704, 4096, 16), (8705, 4096, 0), (8708, 4160, 0)])
def test_conversion_on_both_sides_of_its_lines(rows, K, offset):
    print(f"\n[case] conversion {rows} x {K} offset {offset}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(rows + K)

    def buffer(shape, fill=None):
        n = shape[0] * shape[1]
        whole = torch.full((n + 256,), 0xA5, device="cuda", dtype=torch.uint8)
        if fill is not None:
            whole[offset:offset + n] = fill
        return whole, whole[offset:offset + n].view(shape)

    codes = torch.randint(0, 256, (rows, K // 2), device="cuda", generator=g, dtype=torch.uint8)
    scales = torch.randint(0, 256, (rows, K // 16), device="cuda", generator=g, dtype=torch.uint8)
    want = (codes.view(rows, K // 64, 32).permute(1, 0, 2).reshape(-1), scales.view(rows, K // 64, 4).permute(1, 0, 2).reshape(-1))
    src = [buffer(t.shape, t.reshape(-1)) for t in (codes, scales)]
    there, back = [[buffer(t.shape) for t in (codes, scales)] for _ in range(2)]
    lin, kt = mq.MQ_LAYOUT_LINEAR, mq.MQ_LAYOUT_KTILE
    stream = torch.cuda.current_stream().cuda_stream
    lib = _lib.load()
    for a, b, frm, to in ((src, there, lin, kt), (there, back, kt, lin)):
        assert lib.nvfp4_relayout(a[0][1].data_ptr(), a[1][1].data_ptr(), b[0][1].data_ptr(), b[1][1].data_ptr(), rows, K, frm, to, stream) == 0
    torch.cuda.synchronize()
    for i, t in enumerate((codes, scales)):
        assert torch.equal(there[i][1].view(-1), want[i]) and torch.equal(back[i][1], t)
        for whole, view in (there[i], back[i]):
            assert bool((whole[:offset] == 0xA5).all()) and bool((whole[offset + view.numel():] == 0xA5).all())
