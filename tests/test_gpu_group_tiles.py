"""The tiled group-wise BF6 GEMM, against the oracle.

Its walk over the groups runs ahead of itself (the next group is read and
multiplied while one is folded) over a ring of three stages of 128 codes.  The
shapes have too many output tiles for the few-tile kernel and sit on the edges
of that walk: one, two, three and more stages, a last stage of half a group
pair (K % 128 == 64), an odd and an even number of stages, M and N ragged.
Sums and outputs must equal the oracle's bit for bit: it adds the same rounded
terms in the same order.
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
    (1500, 64, 1401, 64, True), (1473, 128, 1408, 64, False), (1500, 192, 1400, 64, True), (1537, 256, 1399, 64, False),
    (1500, 320, 1404, 64, True), (1409, 384, 1500, 64, False), (1500, 832, 1400, 64, True), (1500, 960, 1433, 64, False),
    (1500, 128, 1401, 128, True), (1473, 256, 1408, 128, False), (1500, 384, 1400, 128, True),
    (1537, 512, 1399, 128, False), (1500, 640, 1404, 128, True), (1409, 896, 1500, 128, False),
]


@pytest.mark.parametrize("M,K,N,G,bias", SHAPES, ids=lambda v: str(v))
def test_tiled_group(M, K, N, G, bias):
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the parity tests need an MI355X")
    print(f"[gpu-group-tiles] {M}x{K}->{N} G={G} bias={bias}", flush=True)
    x_bits = workloads.activations(M, K, "student_t3", 3 * M + N, 0.01, 50.0)
    x_bits[M // 2] = 0
    w_bits = workloads.weights(N, K, 0.02, 3 * M + N + 1)
    b_bits = workloads.bias(N, 0.01, 3 * M + N + 2) if bias else None
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
