"""The int8 engine's kernel on the 6-bit matrix cores (packed operands, many
output tiles, long K).

Its tiles are 256 columns by 6, 7 or 8 bands of 32 rows, it walks K in steps of
256 codes and its loads run two steps ahead, across tiles.  The shapes reach
each height with int4 and with ternary weights: two steps, odd and even
numbers of them, K ending 64, 128 and 192 codes short of a step, one, two and
three tiles per block, M and N ragged, N odd.  Every accumulator and output must
equal the BF6 engine's, and those of rows at the edges of bands and tiles the
oracle's, bit for bit: the contraction is exact.
"""

import numpy as np
import pytest

import oracle
from paper_2609_33601_amd import jq, workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# bands, M, K, N, bias
INT4 = [
    (6, 1287, 256, 5901, True), (6, 3203, 192, 2338, False),  # one step: the int8 kernel
    (6, 4193, 512, 1801, True), (6, 3604, 448, 2054, True),
    (6, 4139, 576, 1852, False), (6, 4168, 640, 1799, True), (6, 8192, 1024, 4104, False),
    (7, 2113, 2240, 5428, True), (7, 2317, 2112, 4877, False), (7, 9216, 2048, 3071, True),
    (8, 4422, 2304, 3081, True), (8, 4088, 2240, 3349, False), (8, 8191, 3072, 4096, True),
]
TERNARY = [
    (6, 4116, 768, 1831, True), (6, 3623, 704, 2061, False), (6, 4101, 2176, 1811, True), (6, 3628, 2112, 2059, True),
    (7, 2121, 2304, 5415, True), (7, 3679, 2240, 3091, False), (7, 5200, 2240, 5201, True),
    (8, 2939, 2304, 4645, True), (8, 4051, 2240, 3384, False), (8, 8191, 3072, 4096, True),
]


@pytest.mark.parametrize("ternary,bands,M,K,N,bias", [(False, *s) for s in INT4] + [(True, *s) for s in TERNARY],
                         ids=lambda v: str(v))
def test_wide(ternary, bands, M, K, N, bias):
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the parity tests need an MI355X")
    print(f"[gpu-gemm-wide] ternary={ternary} {bands} bands: {M}x{K}->{N} bias={bias}", flush=True)
    x_bits = workloads.activations(M, K, "student_t3", 3 * M + N, 0.01, 50.0)
    w_bits = workloads.weights(N, K, 0.02, 3 * M + N + 1)
    b_bits = workloads.bias(N, 0.01, 3 * M + N + 2) if bias else None
    rqx, rsx = oracle.quantize_act(x_bits)
    rwq, rsw = oracle.pack_weight_ternary(w_bits) if ternary else oracle.pack_weight_int4(w_bits)
    b = None if b_bits is None else jq.bf16_tensor(b_bits, "cuda")
    q, s = torch.from_numpy(rqx).cuda(), torch.from_numpy(rsx).cuda()
    wq, sw = torch.from_numpy(rwq).cuda(), torch.from_numpy(rsw).cuda()
    gemm, gemm_i32 = (jq.jq_w158a4_gemm, jq.jq_w158a4_gemm_i32) if ternary else (jq.jq_w4a4_gemm, jq.jq_w4a4_gemm_i32)
    # values behind the outputs must stay as they are
    y = torch.full((M * N + 16,), 7.0, dtype=torch.bfloat16, device="cuda")
    a = torch.full((M * N + 16,), 12345, dtype=torch.int32, device="cuda")
    y4, a4 = y[:M * N].view(M, N), a[:M * N].view(M, N)
    gemm(q, s, wq, sw, b, y4)
    gemm_i32(q, wq, a4)
    wf6 = (jq.jq_ternary_to_f6_weight if ternary else jq.jq_int4_to_f6_weight)(wq)
    xf6 = jq.jq_int4_to_f6(q)
    y6, a6 = torch.empty_like(y4), torch.empty_like(a4)
    jq.jq_w4a4_f6_gemm(xf6, s, K, wf6, sw, b, y6)
    jq.jq_w4a4_f6_gemm_i32(xf6, M, K, wf6, N, a6)
    torch.cuda.synchronize()
    assert torch.equal(a4, a6), "accumulators differ from the BF6 engine's"
    assert torch.equal(y4.view(torch.int16), y6.view(torch.int16)), "outputs differ from the BF6 engine's"
    assert bool((y[M * N:] == 7.0).all()) and bool((a[M * N:] == 12345).all()), "written past the output"

    h = 32 * bands
    rows = sorted({min(max(r, 0), M - 1) for r in (0, 31, 32, h - 1, h, M // h * h - 1, M // 32 * 32, M - 1)})
    acc = (oracle.w158a4_gemm_i32 if ternary else oracle.w4a4_gemm_i32)(rqx[rows], rwq)
    assert np.array_equal(a4[rows].cpu().numpy(), acc), "accumulators differ from the oracle's"
    ref = oracle.epilogue(acc, rsx[rows], rsw, b_bits)
    assert np.array_equal(jq.bf16_bits(y4[rows].contiguous()), ref), "outputs differ from the oracle's"


def test_wide_extreme_codes():
    """The longest K with rows and columns of one code: every product of the offset
    codes at its largest (15 * 15) or smallest, sums up to 225 * 65536 < 2^24."""
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the parity tests need an MI355X")
    M, K, N = 4096, 65536, 4096
    print(f"[gpu-gemm-wide] extreme codes {M}x{K}->{N}", flush=True)
    code = torch.tensor([-8, 7, 0, -1, 1, 3], dtype=torch.int64, device="cuda")
    mc, nc = code[torch.arange(M, device="cuda") % 6], code[torch.arange(N, device="cuda") // 7 % 6]
    pack = lambda c: ((c & 15) * 17).to(torch.uint8)[:, None].expand(-1, K // 2).contiguous()
    a = jq.jq_w4a4_gemm_i32(pack(mc), pack(nc))
    torch.cuda.synchronize()
    assert torch.equal(a.long(), mc[:, None] * nc[None, :] * K), "accumulators differ"


def test_wide_odd_sums_near_the_bound():
    """The longest K with codes close to the largest: sums of the offset codes' products between
    2^23 and 225 * 65536 with their low bits in use, where fp32 has no bit to spare."""
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the parity tests need an MI355X")
    M, K, N = 4096, 65536, 4096
    print(f"[gpu-gemm-wide] near the bound {M}x{K}->{N}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    # row r draws from 7 - r % 4 .. 7
    draw = lambda R: 7 - (torch.rand((R, K), generator=g, device="cuda")
                          * (1 + torch.arange(R, device="cuda") % 4)[:, None]).to(torch.int8)
    pack = lambda c: (c[:, 0::2] | (c[:, 1::2] << 4)).to(torch.uint8)
    cx, cw = draw(M), draw(N)
    a = jq.jq_w4a4_gemm_i32(pack(cx), pack(cw))
    torch.cuda.synchronize()
    sx, sw = cx.sum(1, dtype=torch.int64), cw.sum(1, dtype=torch.int64)
    ref = torch.zeros((M, N), dtype=torch.float64, device="cuda")
    for k in range(0, K, 8192):
        ref += cx[:, k:k + 8192].double() @ cw[:, k:k + 8192].double().t().contiguous()
    ref = ref.long()
    offset = ref + 8 * (sx[:, None] + sw[None, :]) + 64 * K  # what the matrix cores add up
    assert int(offset.min()) > 2 ** 23 and int(offset.max()) > 14.7e6 and len((offset % 64).unique()) == 64
    assert torch.equal(a.long(), ref), "accumulators differ"
