"""The lines between the BF16 product's routes, asked on the host: K slabs of the staged tiles, the decode tile of 112 rows of W,
and which of the two 256x192 tiles runs."""
import pytest

import paper_2605_20315_amd as mq


def _plan(M, N, K, ws):
    parts = mq.mq_bf16_gemm_launches(M, N, K, ws)
    assert len(parts) == 1
    return parts[0]


@pytest.mark.parametrize("M,N,K,most", [
    (65, 4096, 8192, 0), (200, 4096, 8192, 0), (65, 4096, 8256, 10), (200, 4096, 14336, 5), (400, 4096, 14336, 2), (512, 4096, 14336, 2),
    (513, 4096, 14336, 0), (200, 4098, 14336, 0), (200, 4096, 14344, 0), (66, 4, 25600, 33), (2**21 // 4, 4, 8256, 2), (2**21 // 4 + 1, 4, 8256, 0)])
def test_slab_bound_of_the_staged_tiles(M, N, K, most):
    """At most 16 MiB of sums, 768 of K per slab, K above 8192, N % 4 == 0; what is asked for is what is enough."""
    assert mq.mq_bf16_gemm_workspace_bytes(M, N, K) == most * M * N * 4
    slabs = _plan(M, N, K, 64 << 20)["slabs"]
    assert slabs <= max(most, 1) and slabs == _plan(M, N, K, most * M * N * 4)["slabs"]
    assert _plan(M, N, K, 2 * M * N * 4 - 1)["slabs"] == 1


def test_no_slab_is_empty():
    for M in (66, 100, 129, 200, 300, 500):
        for N in (64, 520, 2048, 4096):
            for K in range(8256, 26000, 448):
                steps, slabs = -(-K // 64), _plan(M, N, K, 16 << 20)["slabs"]
                assert K % 64 or (slabs - 1) * -(-steps // slabs) < steps


@pytest.mark.parametrize("M,N,K,tile", [
    (32, 51200, 5120, False), (33, 51200, 5120, True), (48, 51200, 5120, True), (49, 51200, 5120, False), (48, 28672, 4096, True), (48, 4096, 4096, False)])
def test_tile_of_112_rows_of_w(M, N, K, tile):
    assert (_plan(M, N, K, 0)["tile"] == (48, 112)) == tile


@pytest.mark.parametrize("K,kernel", [(192, "bf16_stage"), (448, "bf16_stage"), (512, "bf16_d2l"), (4096, "bf16_d2l")])
def test_256x192_exists_once_per_k(K, kernel):
    seen = {_plan(M, N, K, 0)["kernel"] for M in range(1000, 4200, 97) for N in range(4000, 8000, 331) if _plan(M, N, K, 0)["tile"] == (256, 192)}
    assert seen == {kernel}
