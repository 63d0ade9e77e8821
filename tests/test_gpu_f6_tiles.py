"""The tiled BF6 GEMM at each of its tile heights.

Tiles are 256 columns by 4 (two blocks per CU) or 5, 6, 7 or 8 (one block per
CU) bands of 32 rows; the shape decides which.  Per height: one, two and more
tiles per block; tiles of one, two and three stages of 128 codes, of an odd
and of an even number; M and N ragged against the tile, N odd (element-wise
stores, the bias' last value on its own), N a multiple of 8 only.
Every output and accumulator must equal the int8 engine's, and those of rows
at the edges of bands and tiles the oracle's, bit for bit: the contraction is
exact and the epilogue's rounding steps are the oracle's.
"""

import numpy as np
import pytest

import oracle
from paper_2609_33601_amd import jq, workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# bands, M, K, N, bias
SHAPES = [
    (4, 1056, 128, 1241, True), (4, 5457, 256, 2819, False), (4, 5401, 384, 5907, True), (4, 4225, 640, 4680, True),
    (5, 5387, 128, 1285, True), (5, 5427, 256, 1352, True), (5, 5422, 320, 1295, False), (5, 5400, 1088, 2819, True),
    (5, 5022, 3072, 3078, True),
    (6, 5925, 576, 1577, True), (6, 4366, 640, 5552, False), (6, 5891, 3072, 5391, True), (6, 4378, 3008, 5384, True),
    (7, 5398, 1664, 4360, True), (7, 4225, 1856, 5640, True), (7, 4909, 3008, 4913, False),
    (8, 2693, 3008, 4865, True), (8, 5853, 3072, 4616, False), (8, 4096, 3200, 4096, True),
]


@pytest.mark.parametrize("bands,M,K,N,bias", SHAPES, ids=lambda v: str(v))
def test_tile_height(bands, M, K, N, bias):
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the parity tests need an MI355X")
    print(f"[gpu-f6-tiles] {bands} bands: {M}x{K}->{N} bias={bias}", flush=True)
    x_bits = workloads.activations(M, K, "student_t3", 3 * M + N, 0.01, 50.0)
    w_bits = workloads.weights(N, K, 0.02, 3 * M + N + 1)
    b_bits = workloads.bias(N, 0.01, 3 * M + N + 2) if bias else None
    rwq, rsw = oracle.pack_weight_int4(w_bits)
    rqx, rsx = oracle.quantize_act(x_bits)

    b = None if b_bits is None else jq.bf16_tensor(b_bits, "cuda")
    wq, qx = torch.from_numpy(rwq).cuda(), torch.from_numpy(rqx).cuda()
    sw, sx = torch.from_numpy(rsw).cuda(), torch.from_numpy(rsx).cuda()
    wf6, xf6 = jq.jq_int4_to_f6_weight(wq), jq.jq_int4_to_f6(qx)
    # the values past the outputs must stay as they are
    y = torch.full((M * N + 16,), 7.0, dtype=torch.bfloat16, device="cuda")
    a = torch.full((M * N + 16,), 12345, dtype=torch.int32, device="cuda")
    y6, a6 = y[:M * N].view(M, N), a[:M * N].view(M, N)
    jq.jq_w4a4_f6_gemm(xf6, sx, K, wf6, sw, b, y6)
    jq.jq_w4a4_f6_gemm_i32(xf6, M, K, wf6, N, a6)
    y4 = jq.jq_w4a4_gemm(qx, sx, wq, sw, b)
    a4 = jq.jq_w4a4_gemm_i32(qx, wq)
    torch.cuda.synchronize()
    assert torch.equal(a6, a4), "accumulators differ from the int8 engine's"
    assert torch.equal(y6.view(torch.int16), y4.view(torch.int16)), "outputs differ from the int8 engine's"
    assert bool((y[M * N:] == 7.0).all()) and bool((a[M * N:] == 12345).all()), "written past the output"

    edges = [0, 31, 32, 32 * bands - 1, 32 * bands, 64 * bands - 1, M // (32 * bands) * 32 * bands - 1, M // 32 * 32, M - 1]
    rows = sorted({min(max(r, 0), M - 1) for r in edges})
    acc = oracle.w4a4_gemm_i32(rqx[rows], rwq)
    ref = oracle.w4a4_gemm(rqx[rows], rsx[rows], rwq, rsw, b_bits)
    assert np.array_equal(a6[rows].cpu().numpy(), acc), "accumulators differ from the oracle's"
    assert np.array_equal(jq.bf16_bits(y6[rows].contiguous()), ref), "outputs differ from the oracle's"
