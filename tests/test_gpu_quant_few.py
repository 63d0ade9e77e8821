"""The BF6 quantisers' few-row kernel against the four-row and the long-row kernels.

An input of up to 512 rows of up to 16384 codes takes the few-row kernel (of
longer rows, fewer: see f6_quantize_few_rows), one of more rows the
others, whose codes and scales the oracle tests pin.  The first rows of a
longer input must therefore come out byte for byte as they do alone, padding
included: operand bytes and scale bits, per token and per group, for row
lengths at the kernel's edges (a part of a wave, one chunk per thread, a K
tail, the longest register-resident row, rows of several chunks per thread),
with rows that take its special paths (zeros, exact ties, a reciprocal that
overflows, infinities and NaN).  The batched form must equal single calls, on
both of its kernels.
"""

import numpy as np
import pytest

from paper_2609_33601_amd import jq, workloads
from tests.routes import few_rows, few_rows_batch

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _rows(M, K, seed):
    bits = workloads.activations(M, K, "student_t3", seed, 0.01, 50.0)
    bits[0] = 0                                  # scale zero
    if M > 3:
        bits[1] = 0x3F80                         # all one: every code 7
        bits[1, 1::2] = 0x3F00                   # halves: 3.5, a tie
        bits[2] &= 0x81FF                        # tiny values: the reciprocal overflows
        bits[3, K // 2] = 0x7F80                 # an infinity
    if M > 5:
        bits[4, 1] = 0x7FC0                      # a NaN
    return bits


@pytest.mark.parametrize("G", [0, 64, 128])
@pytest.mark.parametrize("M,K", [(1, 64), (2, 128), (33, 192), (512, 256), (7, 3072), (96, 4096), (64, 4160),
                                 (31, 12288), (5, 16384), (3, 16448), (6, 20480), (2, 32832), (4, 65536),
                                 (33, 16448), (40, 20480), (4, 20480), (4, 49152), (32, 32832), (48, 49152), (160, 65536)],
                         ids=lambda v: str(v))
def test_few_rows_equal_many(M, K, G):
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    if G and K % G:
        pytest.skip("not a multiple of the group")
    print(f"[gpu-quant-few] {M}x{K} G={G} few={few_rows(M, K, G)}", flush=True)
    assert not few_rows(544, K, G)
    x = torch.zeros((544, K), dtype=torch.bfloat16, device="cuda")
    x[:M] = jq.bf16_tensor(_rows(M, K, M + K), "cuda")
    f = (lambda t: jq.jq_quantize_act_group_f6(t, G)) if G else jq.jq_quantize_act_f6
    big, bs = f(x)
    n = jq.jq_f6_operand_bytes(M, K)
    q = torch.full((n + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    s = torch.full((M * (K // G if G else 1) + 16,), 7.0, device="cuda")
    sv = s[:-16].view(M, K // G) if G else s[:-16]
    few = x[:M].contiguous()
    if G:
        jq.jq_quantize_act_group_f6(few, G, q[:n], sv)
    else:
        jq.jq_quantize_act_f6(few, q[:n], sv)
    torch.cuda.synchronize()
    assert torch.equal(q[:n], big[:n]), "operand bytes differ"
    assert torch.equal(sv.contiguous().view(torch.int32), bs[:M].contiguous().view(torch.int32)), "scales differ"
    assert bool((q[n:] == 0xA5).all()) and bool((s[-16:] == 7.0).all()), "written past the outputs"


@pytest.mark.parametrize("shapes", [[(1, 64)], [(64, 4096), (3, 12288), (40, 256)], [(5, 20480), (512, 192), (1, 65536)],
                                    [(9, 3072), (700, 128)], [(512, 4096), (512, 4096), (300, 1024), (512, 12288)]], ids=str)
def test_few_rows_batch(shapes):
    print("[gpu-quant-few] batch", shapes, "few", few_rows_batch(shapes), flush=True)
    xs = [jq.bf16_tensor(_rows(M, K, i), "cuda") for i, (M, K) in enumerate(shapes)]
    qs, ss = jq.jq_quantize_act_f6_batch(xs)
    for x, q, s in zip(xs, qs, ss):
        q1, s1 = jq.jq_quantize_act_f6(x)
        assert np.array_equal(q.cpu().numpy(), q1.cpu().numpy())
        assert torch.equal(s.view(torch.int32), s1.view(torch.int32))
