"""The group-wise BF6 GEMM's kernel for products with few output tiles, against the oracle.

Its tile is 32 x 32, its four or eight waves take one unit of 128 codes each
per round, and every output's group terms are added in k order.  The shapes
sit on the edges: one row, a few columns, one past a band, odd N, K of fewer
units than waves, of a last round that is not full and (G = 64) ends in half a
unit; with either number of waves, and just past the line on the tiled kernel
(ragged; K of one group, of one unit).  Sums and outputs must equal the oracle's
bit for bit: every fp32 step of the layer is rounded on its own, in a fixed
order.  A row of zeros, whose scales are zero, stays the bias.
"""

import numpy as np
import pytest

import oracle
from oracle import group_sum_c
from paper_2609_33601_amd import jq, workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# M, K, N, G, bias
SHAPES = [
    (1, 64, 1, 64, True), (1, 128, 2, 128, True), (32, 192, 31, 64, False), (33, 1088, 999, 64, True),
    (2, 12288, 6, 64, True), (3, 4096, 4095, 128, False),
    (33, 4096, 12287, 128, True), (70, 1152, 5001, 64, True), (129, 3200, 4098, 128, False), (40, 640, 8200, 64, False),
    (700, 512, 6001, 128, True), (1100, 320, 4097, 64, True),
]


@pytest.mark.parametrize("M,K,N,G,bias", SHAPES, ids=lambda v: str(v))
def test_few_tiles_group(M, K, N, G, bias):
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the parity tests need an MI355X")
    print(f"[gpu-group-narrow] {M}x{K}->{N} G={G} bias={bias}", flush=True)
    x_bits = workloads.activations(M, K, "student_t3", 5 * M + N, 0.01, 50.0)
    x_bits[M // 2] = 0
    w_bits = workloads.weights(N, K, 0.02, 5 * M + N + 1)
    b_bits = workloads.bias(N, 0.01, 5 * M + N + 2) if bias else None
    rwq, rsw = oracle.pack_weight_int4_group(w_bits, G)
    rqx, rsx = oracle.quantize_act_group(x_bits, G)
    rs = group_sum_c.w4a4g_gemm_f32(rqx, rsx, rwq, rsw, G)
    ref = oracle.group_epilogue(rs, b_bits)

    b = None if b_bits is None else jq.bf16_tensor(b_bits, "cuda")
    wf6 = jq.jq_int4_to_f6_weight(torch.from_numpy(rwq).cuda())
    xf6 = jq.jq_int4_to_f6(torch.from_numpy(rqx).cuda())
    sw, sx = torch.from_numpy(rsw).cuda(), torch.from_numpy(rsx).cuda()
    # values behind the outputs must stay as they are
    y = torch.full((M * N + 16,), 7.0, dtype=torch.bfloat16, device="cuda")
    s = torch.full((M * N + 16,), 7.0, dtype=torch.float32, device="cuda")
    jq.jq_w4a4g_f6_gemm(xf6, sx, wf6, sw, G, b, y[:M * N].view(M, N))
    jq.jq_w4a4g_f6_gemm_f32(xf6, sx, wf6, sw, G, s[:M * N].view(M, N))
    torch.cuda.synchronize()
    got = s[:M * N].view(M, N).cpu().numpy()
    assert np.array_equal(got.view(np.uint32), rs.view(np.uint32)), "group sums differ"
    d = int(np.count_nonzero(jq.bf16_bits(y[:M * N].view(M, N)) != ref))
    assert d == 0, f"{d} of {M * N} outputs differ"
    assert bool((y[M * N:] == 7.0).all()) and bool((s[M * N:] == 7.0).all()), "written past the output"
