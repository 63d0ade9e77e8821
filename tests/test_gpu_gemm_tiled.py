"""The packed engine's int8 kernel at both of its tile heights, in both weight formats.

Its tiles are 128 or 112 rows by 256 columns and it walks K in stages of 128
codes.  Products with few tiles, and large ones with long K, go to kernels of
their own; the shapes are what is left: per format and height an even K and one
that ends in half a stage, M and N ragged, N odd, a multiple of 2 and of 8.
Every accumulator and output, with and without a bias, must equal the BF6
engine's, and those of rows at the edges of fragments and tiles the oracle's,
bit for bit: the contraction is exact.
"""

import numpy as np
import pytest

import oracle
from paper_2609_33601_amd import jq, workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# tile rows, M, K, N
INT4 = [
    (128, 3981, 512, 1915), (128, 4090, 384, 8192), (128, 1262, 320, 5917), (128, 1917, 576, 3806),
    (112, 4608, 512, 9216), (112, 9215, 640, 3071), (112, 1147, 192, 8958), (112, 2300, 448, 3001),
]
TERNARY = [
    (128, 3981, 512, 1915), (128, 4090, 384, 8192), (128, 1262, 320, 5917), (128, 1917, 576, 3806),
    (112, 4608, 512, 9216), (112, 9215, 640, 3071), (112, 2583, 896, 2150), (112, 2270, 448, 4415),
]


@pytest.mark.parametrize("ternary,height,M,K,N", [(False, *s) for s in INT4] + [(True, *s) for s in TERNARY],
                         ids=lambda v: str(v))
def test_tiled(ternary, height, M, K, N):
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the parity tests need an MI355X")
    print(f"[gpu-gemm-tiled] ternary={ternary} {height} rows: {M}x{K}->{N}", flush=True)
    x_bits = workloads.activations(M, K, "student_t3", 3 * M + N, 0.01, 50.0)
    w_bits = workloads.weights(N, K, 0.02, 3 * M + N + 1)
    b_bits = workloads.bias(N, 0.01, 3 * M + N + 2)
    rqx, rsx = oracle.quantize_act(x_bits)
    rwq, rsw = oracle.pack_weight_ternary(w_bits) if ternary else oracle.pack_weight_int4(w_bits)
    b = jq.bf16_tensor(b_bits, "cuda")
    q, s = torch.from_numpy(rqx).cuda(), torch.from_numpy(rsx).cuda()
    wq, sw = torch.from_numpy(rwq).cuda(), torch.from_numpy(rsw).cuda()
    gemm, gemm_i32 = (jq.jq_w158a4_gemm, jq.jq_w158a4_gemm_i32) if ternary else (jq.jq_w4a4_gemm, jq.jq_w4a4_gemm_i32)
    # values behind the outputs must stay as they are
    a = torch.full((M * N + 16,), 12345, dtype=torch.int32, device="cuda")
    yv = [torch.full((M * N + 16,), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    outs, a4 = [t[:M * N].view(M, N) for t in yv], a[:M * N].view(M, N)
    for bias, out in zip((b, None), outs):
        gemm(q, s, wq, sw, bias, out)
    gemm_i32(q, wq, a4)
    wf6 = (jq.jq_ternary_to_f6_weight if ternary else jq.jq_int4_to_f6_weight)(wq)
    xf6 = jq.jq_int4_to_f6(q)
    ref6 = [jq.jq_w4a4_f6_gemm(xf6, s, K, wf6, sw, bias) for bias in (b, None)]
    a6 = jq.jq_w4a4_f6_gemm_i32(xf6, M, K, wf6, N)
    torch.cuda.synchronize()
    assert torch.equal(a4, a6), "accumulators differ from the BF6 engine's"
    for out, ref in zip(outs, ref6):
        assert torch.equal(out.view(torch.int16), ref.view(torch.int16)), "outputs differ from the BF6 engine's"
    assert all(bool((t[M * N:] == 7.0).all()) for t in yv) and bool((a[M * N:] == 12345).all()), "written past the output"

    edges = (0, 15, 16, height - 1, height, M // height * height - 1, M // 16 * 16, M - 1)
    rows = sorted({min(max(r, 0), M - 1) for r in edges})
    acc = (oracle.w158a4_gemm_i32 if ternary else oracle.w4a4_gemm_i32)(rqx[rows], rwq)
    assert np.array_equal(a4[rows].cpu().numpy(), acc), "accumulators differ from the oracle's"
    for out, bits in zip(outs, (b_bits, None)):
        ref = oracle.epilogue(acc, rsx[rows], rsw, bits)
        assert np.array_equal(jq.bf16_bits(out[rows].contiguous()), ref), "outputs differ from the oracle's"
