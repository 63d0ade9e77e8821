"""The packed-int4 GEMM's kernel for products with few output tiles, against the oracle.

Its tiles are 32x32, 64x64 and 64x96, its four waves split K in units of 128
codes (256 with ternary weights) and each lane group takes a quarter of a
unit.  The shapes sit on the edges: one row or column, one past 16 and 32, N
not a multiple of 4 (element-wise stores), K of a part of a unit, of fewer
units than waves, of an odd number of units; each tile, both weight formats;
and ragged shapes just past the line, on the tiled kernel.  Accumulators and
outputs must equal the oracle's bit for bit (exact integers, and the oracle's
rounding steps in the epilogue).
"""

import numpy as np
import pytest

import oracle
from paper_2609_33601_amd import jq, workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# M, K, N, bias
SHAPES = [
    (1, 64, 1, True), (17, 128, 33, False), (32, 192, 30, True), (65, 1024, 999, True), (33, 4096, 3001, False),
    (1, 12288, 4, False), (33, 320, 12286, True), (64, 4160, 8190, False), (300, 3136, 3003, True),
    (97, 3072, 12285, True), (500, 1088, 3072, False),
    (1100, 1088, 3077, True), (2300, 448, 3001, True),  # the tiled kernel
]


@pytest.mark.parametrize("ternary", [False, True], ids=["int4", "ternary"])
@pytest.mark.parametrize("M,K,N,bias", SHAPES, ids=lambda v: str(v))
def test_few_tiles_int8(M, K, N, bias, ternary):
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the parity tests need an MI355X")
    print(f"[gpu-gemm-narrow] {M}x{K}->{N} bias={bias} ternary={ternary}", flush=True)
    x_bits = workloads.activations(M, K, "student_t3", 3 * M + N, 0.01, 50.0)
    w_bits = workloads.weights(N, K, 0.02, 3 * M + N + 1)
    b_bits = workloads.bias(N, 0.01, 3 * M + N + 2) if bias else None
    rqx, rsx = oracle.quantize_act(x_bits)
    if ternary:
        rwq, rsw = oracle.pack_weight_ternary(w_bits)
        acc = oracle.w158a4_gemm_i32(rqx, rwq)
        ref = oracle.w158a4_linear(x_bits, rwq, rsw, b_bits)
        gemm, gemm_i32 = jq.jq_w158a4_gemm, jq.jq_w158a4_gemm_i32
    else:
        rwq, rsw = oracle.pack_weight_int4(w_bits)
        acc = oracle.w4a4_gemm_i32(rqx, rwq)
        ref = oracle.w4a4_gemm(rqx, rsx, rwq, rsw, b_bits)
        gemm, gemm_i32 = jq.jq_w4a4_gemm, jq.jq_w4a4_gemm_i32

    b = None if b_bits is None else jq.bf16_tensor(b_bits, "cuda")
    q, s = torch.from_numpy(rqx).cuda(), torch.from_numpy(rsx).cuda()
    wq, sw = torch.from_numpy(rwq).cuda(), torch.from_numpy(rsw).cuda()
    # values behind the outputs must stay as they are
    y = torch.full((M * N + 16,), 7.0, dtype=torch.bfloat16, device="cuda")
    a = torch.full((M * N + 16,), 12345, dtype=torch.int32, device="cuda")
    gemm(q, s, wq, sw, b, y[:M * N].view(M, N))
    gemm_i32(q, wq, a[:M * N].view(M, N))
    torch.cuda.synchronize()
    assert np.array_equal(a[:M * N].view(M, N).cpu().numpy(), acc), "accumulators differ"
    d = int(np.count_nonzero(jq.bf16_bits(y[:M * N].view(M, N)) != ref))
    assert d == 0, f"{d} of {M * N} outputs differ"
    assert bool((y[M * N:] == 7.0).all()) and bool((a[M * N:] == 12345).all()), "written past the output"
