"""The BF6 GEMM's kernel for products with few output tiles, against the oracle.

Its tiles are 1x1, 1x2, 2x2 and 2x3 bands of 32 rows x 32 columns, its four
waves split K in units of 128 codes and it loads two units ahead.  The shapes
sit on the edges of these: one row or column, one past a band, a tile's last
band or column absent, N not a multiple of 4 (element-wise stores), K of one
unit, of half a unit, of less than a unit per wave, of an odd number of units
per wave.  They cover each of its tiles (the rules' estimates decide which), and
three ragged shapes just past the line, on the tiled kernel with one block per
CU and with two.
Accumulators and outputs must equal the oracle's bit for bit: the contraction
is exact in any order and the epilogue's rounding steps are the oracle's.
"""

import numpy as np
import pytest

import oracle
from paper_2609_33601_amd import jq, workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# M, K, N, bias
SHAPES = [
    (1, 64, 1, True), (32, 64, 30, False), (31, 192, 33, True), (65, 1024, 999, True), (33, 4096, 4095, False),
    (1, 12288, 4, False), (3, 3072, 12288, False),                     # 1x1
    (96, 12288, 4097, True),                                           # 1x2
    (300, 12288, 3000, True), (64, 4096, 12288, False), (40, 4160, 12287, True),  # 2x2
    (97, 3072, 12285, True), (512, 3072, 3072, False),                 # 2x3
    (1500, 6272, 5000, True), (2300, 6208, 3001, True), (777, 320, 12286, True),  # the tiled kernel
]


@pytest.mark.parametrize("M,K,N,bias", SHAPES, ids=lambda v: str(v))
def test_few_tiles(M, K, N, bias):
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the parity tests need an MI355X")
    print(f"[gpu-f6-narrow] {M}x{K}->{N} bias={bias}", flush=True)
    x_bits = workloads.activations(M, K, "student_t3", 7 * M + N, 0.01, 50.0)
    w_bits = workloads.weights(N, K, 0.02, 7 * M + N + 1)
    b_bits = workloads.bias(N, 0.01, 7 * M + N + 2) if bias else None
    rwq, rsw = oracle.pack_weight_int4(w_bits)
    rqx, rsx = oracle.quantize_act(x_bits)
    acc = oracle.w4a4_gemm_i32(rqx, rwq)
    ref = oracle.w4a4_gemm(rqx, rsx, rwq, rsw, b_bits)

    b = None if b_bits is None else jq.bf16_tensor(b_bits, "cuda")
    wf6 = jq.jq_int4_to_f6_weight(torch.from_numpy(rwq).cuda())
    xf6 = jq.jq_int4_to_f6(torch.from_numpy(rqx).cuda())
    sw, sx = torch.from_numpy(rsw).cuda(), torch.from_numpy(rsx).cuda()
    # rows and columns around the outputs, which must stay as they are
    y = torch.full((M * N + 16,), 7.0, dtype=torch.bfloat16, device="cuda")
    a = torch.full((M * N + 16,), 12345, dtype=torch.int32, device="cuda")
    jq.jq_w4a4_f6_gemm(xf6, sx, K, wf6, sw, b, y[:M * N].view(M, N))
    jq.jq_w4a4_f6_gemm_i32(xf6, M, K, wf6, N, a[:M * N].view(M, N))
    torch.cuda.synchronize()
    assert np.array_equal(a[:M * N].view(M, N).cpu().numpy(), acc), "accumulators differ"
    d = int(np.count_nonzero(jq.bf16_bits(y[:M * N].view(M, N)) != ref))
    assert d == 0, f"{d} of {M * N} outputs differ"
    assert bool((y[M * N:] == 7.0).all()) and bool((a[M * N:] == 12345).all()), "written past the output"
