"""The tensor-level scale at the sizes where its launch changes: one workgroup of 64 KB shares up to four of them, workgroups
that count themselves up to 96, a launch of its own for the last step beyond.  Exact: a maximum and one IEEE division."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_20315_amd as mq

from _gpu_util import dev_bf16

pytestmark = pytest.mark.gpu

SHARE = 32768  # elements a workgroup takes
# (rows, K): 0, 1 and 16 elements, 4 shares and a row more, 96 shares and a row more, 128, 256 and more
SIZES = [(0, 64), (1, 16), (3, 48), (4 * SHARE // 64, 64), (4 * SHARE // 64 + 1, 64), (96 * SHARE // 4096, 4096),
         (96 * SHARE // 4096 + 1, 4096), (128 * SHARE // 4096, 4096),
         (128 * SHARE // 4096 + 1, 4096), (256 * SHARE // 4096 + 1, 4096), (977, 14336)]


@pytest.mark.parametrize("rows,K", SIZES)
@pytest.mark.parametrize("pad", [0, 8])
def test_scale_against_oracle(rows, K, pad):
    print(f"\n[case] global scale rows={rows} K={K} pad={pad}", flush=True)
    rng = np.random.default_rng([rows, K])
    x = rng.integers(0, 0x3F80, size=(rows, K + pad)).astype(np.uint16) | (rng.integers(0, 2, size=(rows, K + pad)) << 15).astype(np.uint16)
    x[:, K:] = 0x7F00                                            # beyond the rows: larger than anything in them
    xd = dev_bf16(x)[:, :K] if rows else torch.empty((0, K), dtype=torch.bfloat16, device="cuda")
    out = torch.full((1,), 3.0e38, device="cuda")                # what an earlier call may have left
    places = [(0, 0), (rows - 1, K - 1), (rows // 2, K // 3)] if rows else [None]
    for i, at in enumerate(places):                              # the largest value: first, last, in between; rising
        if at:
            x[at] = 0xC000 + i
            xd[at] = torch.tensor([0xC000 + i - 0x10000], dtype=torch.int16, device="cuda").view(torch.bfloat16)[0]
        want = oracle.global_scale(np.ascontiguousarray(x[:, :K])) if rows else np.float32(1.0)
        got = mq.nvfp4_global_scale(xd, out)
        assert np.float32(got.item()) == want
    if rows:
        xd.zero_()
        assert mq.nvfp4_global_scale(xd, out).item() == 1.0


@pytest.mark.parametrize("rows", [16, 512, 4096])
def test_scale_replayed_from_a_graph(rows):
    K = 4096
    mq.mq_init()
    x = torch.zeros(rows, K, dtype=torch.bfloat16, device="cuda")
    out = torch.zeros(1, device="cuda")
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        mq.nvfp4_global_scale(x, out)
    for i in range(6):
        x.normal_(std=float(2 ** (3 - i)))
        graph.replay()
        torch.cuda.synchronize()
        eager = mq.nvfp4_global_scale(x, torch.empty(1, device="cuda"))
        assert out.item() == eager.item() == float(np.float32(x.abs().max().float().item()) / np.float32(2688.0))
