"""The gate's calls at the edges of their kernels (expert tiles, token tiles, remainders of the hidden dimension),
against 64-bit arithmetic.

Logits: fp32 sums of d products of N(0,1) x N(0,0.02) values, each off by at most d * 2^-24 of the sum of the absolute
products; 1e-5 of the logits' scale is what the stage tests allow as well.
"""
import numpy as np
import pytest
import torch

from paper_2602_11686_amd import binding as B

pytestmark = pytest.mark.gpu


def gate_case(T, d, E, k, dtype, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.empty(T, d, dtype=dtype, device="cuda").normal_(generator=g)
    wg = torch.empty(d, E, dtype=dtype, device="cuda").normal_(0.0, 0.02, generator=g)
    bias = torch.empty(E, dtype=torch.float32, device="cuda").normal_(0.0, 0.1, generator=g)
    s = B.Shape(T, d, 8, E, k, dtype)
    ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    out = (torch.full((T, k), -7, dtype=torch.int32, device="cuda"), torch.empty(T, k, device="cuda"),
           torch.full((T, E), float("nan"), device="cuda"))
    return s, x, wg, bias, ws, out


SIZES = [(1, 36, 1, 1, torch.float32), (15, 4, 16, 16, torch.float32), (17, 260, 17, 3, torch.float32),
         (33, 132, 65, 4, torch.float32), (70, 1024, 130, 8, torch.float32), (40, 516, 256, 8, torch.float32),
         (1, 8, 2, 2, torch.bfloat16), (31, 264, 33, 5, torch.bfloat16), (50, 1096, 200, 8, torch.bfloat16),
         (1, 256, 8, 2, torch.bfloat16), (33, 512, 256, 8, torch.bfloat16), (64, 2048, 128, 8, torch.bfloat16),
         # the ends of the range in which the hidden dimension is split over workgroups, and past them
         (1024, 256, 20, 4, torch.bfloat16), (1025, 256, 20, 4, torch.bfloat16), (2048, 132, 9, 2, torch.float32),
         (2049, 132, 9, 2, torch.float32), (2050, 264, 33, 2, torch.bfloat16),
         (905, 768, 200, 8, torch.bfloat16), (2000, 264, 129, 2, torch.float32)]  # 57 and 125 token tiles: no even split of 256


# bf16 kernels that contract the whole hidden dimension: one to 16 expert tiles, 16 and 32 tokens per workgroup with a remainder,
# four and eight parts of the hidden dimension, of one chunk (half a pair) and of several
SIZES += [(1030, d, E, k, torch.bfloat16) for d, E, k in [(256, 3, 2), (512, 17, 3), (768, 40, 2), (2560, 16, 4), (768, 100, 8), (256, 200, 6)]]
SIZES += [(8191, 256, 20, 2, torch.bfloat16), (8192, 512, 32, 2, torch.bfloat16), (8205, 256, 50, 2, torch.bfloat16), (8205, 512, 50, 2, torch.bfloat16),
          # hidden dimensions that are no multiple of 256, past the batches whose dimension is split: the packed weight of the fp32 MFMAs
          (2050, 1096, 24, 3, torch.bfloat16), (2060, 520, 200, 8, torch.bfloat16), (2049, 2056, 100, 4, torch.bfloat16), (2049, 648, 3, 1, torch.bfloat16),
          # as many experts as the tiles hold: a lane reads those of a k-row at once; split and not, with a remainder of k
          (100, 1032, 32, 3, torch.bfloat16), (33, 72, 64, 2, torch.bfloat16), (700, 520, 128, 8, torch.bfloat16), (2049, 264, 64, 4, torch.bfloat16),
          (8205, 768, 9, 2, torch.bfloat16), (16383, 256, 128, 3, torch.bfloat16), (16401, 256, 128, 3, torch.bfloat16)]


# the packed weight on either side of its lines: one tile of experts, 16 of 17, 5 of 8, 9 of 16, 3 of 4, 6 of 8, the 2 tiles that 32 experts
# fill, 7 of 8
PACKED = [(2049, 904, 7, 2), (2049, 760, 7, 2), (2901, 648, 7, 2), (2051, 520, 20, 2), (3900, 2056, 70, 2), (2060, 1096, 70, 2), (4097, 520, 130, 2), (2049, 520, 130, 2),
          (2049, 904, 40, 2), (2049, 904, 90, 2), (2049, 520, 90, 2), (2049, 3080, 32, 2), (2049, 1096, 32, 2), (2310, 520, 100, 2), (2049, 520, 100, 2)]
SIZES += [(T, d, E, k, torch.bfloat16) for T, d, E, k in PACKED]


@pytest.mark.parametrize("T,d,E,k", PACKED)
def test_gate_weight_forms_give_the_same_bits(T, d, E, k):
    """Packed or not, which goes by the sizes and by the workspace that the caller brings."""
    s, x, wg, bias, ws, out = gate_case(T, d, E, k, torch.bfloat16, T + E)
    B.moe_gate_topk(s, x, wg, bias, *out, ws)
    other = [torch.empty_like(v) for v in out]
    B.moe_gate_topk(s, x, wg, bias, *other, ws[:0])
    torch.cuda.synchronize()
    assert all(torch.equal(u, v) for u, v in zip(out, other))


@pytest.mark.parametrize("least_ws", [False, True])  # with the least workspace the dimension is never split
@pytest.mark.parametrize("T,d,E,k,dtype", SIZES)
def test_gate_topk_edges(T, d, E, k, dtype, least_ws):
    s, x, wg, bias, ws, (ids, w, logits) = gate_case(T, d, E, k, dtype, T + d + E)
    if least_ws:
        ws = ws[:512 * d] if dtype == torch.bfloat16 and d % 256 == 0 else ws[:0]
    B.moe_gate_topk(s, x, wg, bias, ids, w, logits, ws)
    want = x.double() @ wg.double() + bias.double()
    scale = max(1.0, float(want.abs().max()))
    assert float((logits.double() - want).abs().max()) <= 1e-5 * scale
    # the picks are the sorted top-k of the logits that the call returned, lower index first among equals
    order = np.argsort(-logits.cpu().numpy(), axis=1, kind="stable")[:, :k]
    np.testing.assert_array_equal(ids.cpu().numpy(), order)
    ref_w = torch.softmax(want.gather(1, ids.long()), 1)
    assert float((w.double() - ref_w).abs().max()) <= 1.2e-5


@pytest.mark.parametrize("d,dtype", [(36, torch.float32), (264, torch.bfloat16), (256, torch.bfloat16)])
def test_gate_topk_with_nan_and_equal_logits(d, dtype):
    """Equal columns: lower expert first.  A token without a comparable logit still gets indices in range."""
    s, x, wg, bias, ws, (ids, w, logits) = gate_case(20, d, 6, 3, dtype, 5)
    wg[:] = wg[:, :1]
    bias.zero_()
    x[7] = float("nan")
    B.moe_gate_topk(s, x, wg, bias, ids, w, logits, ws)
    got = ids.cpu().numpy()
    assert ((got >= 0) & (got < 6)).all()
    for t in range(20):
        if t != 7:
            assert got[t].tolist() == [0, 1, 2]


@pytest.mark.parametrize("T,d,E,k,dtype", [(1, 36, 5, 2, torch.float32), (33, 68, 65, 3, torch.float32),
                                           (700, 128, 8, 2, torch.float32), (300, 1028, 256, 8, torch.float32),
                                           (9000, 68, 3, 2, torch.float32)])  # more chunks of tokens than a workgroup has threads
def test_gate_bwd_edges(T, d, E, k, dtype):
    s, x, wg, bias, ws, (ids, w, logits) = gate_case(T, d, E, k, dtype, 3 * T + E)
    B.moe_gate_topk(s, x, wg, bias, ids, w, None, ws)
    g = torch.Generator(device="cuda").manual_seed(1)
    dw = torch.empty(T, k, device="cuda").normal_(generator=g)
    dx = torch.empty(T, d, dtype=dtype, device="cuda").normal_(generator=g)
    dx0, dwg = dx.double(), torch.full((d, E), float("nan"), device="cuda")
    B.moe_gate_topk_bwd(s, x, wg, ids, w, dw, dx, dwg, ws)
    wd, dwd = w.double(), dw.double()
    dl = torch.zeros(T, E, dtype=torch.float64, device="cuda").scatter_(
        1, ids.long(), wd * (dwd - (wd * dwd).sum(1, keepdim=True)))
    ref = x.double().t() @ dl
    # fp32 sums of T products: 2^-24 each, partly cancelling; 1e-5 of the largest is 170 roundings of the whole sum
    assert float((dwg.double() - ref).abs().max()) <= 1e-5 * float(ref.abs().max())
    ref = dx0 + dl @ wg.double().t()
    assert float((dx.double() - ref).abs().max()) <= 1e-5 * float(ref.abs().max())


def test_gate_topk_more_tokens_than_a_grid_dimension():
    """2^27 tokens are 2^23 workgroups of 512 threads.  Two experts, top-1; fp32 logits of four terms of magnitude <= 1 are
    within 2^-22 of the exact ones."""
    T, d, E = (1 << 27) + 33, 4, 2
    g = torch.Generator(device="cuda").manual_seed(2)
    x = torch.empty(T, d, device="cuda").uniform_(-1.0, 1.0, generator=g)
    wg = torch.tensor([[1.0, -0.5], [0.25, 1.0], [-1.0, 0.5], [0.75, -1.0]], device="cuda")
    ids, w = torch.full((T, 1), -7, dtype=torch.int32, device="cuda"), torch.full((T, 1), float("nan"), device="cuda")
    B.moe_gate_topk(B.Shape(T, d, 4, E, 1, torch.float32), x, wg, None, ids, w, None,
                    torch.empty(0, dtype=torch.uint8, device="cuda"))
    v = (wg[:, 0] - wg[:, 1]).double()
    for i in range(0, T, 1 << 24):  # (in parts: the library's product over all of them is not to be relied on)
        gap = (x[i:i + (1 << 24)].double() * v).sum(1)
        got, want = ids[i:i + (1 << 24), 0], (gap < 0).to(torch.int32)
        assert bool(((got == want) | (gap.abs() < 1e-5)).all()), i
        assert int(got.min()) >= 0 and int(got.max()) <= 1 and bool((w[i:i + (1 << 24)] == 1.0).all()), i


def test_gate_bwd_more_tokens_than_a_grid_dimension():
    """2^26 tokens are 2^24 workgroups of 256 threads in the launch that expands dL."""
    T, d, E, k = (1 << 26) + 1029, 4, 3, 2
    g = torch.Generator(device="cuda").manual_seed(3)
    s = B.Shape(T, d, 4, E, k, torch.float32)
    x = torch.empty(T, d, device="cuda").normal_(generator=g)
    wg = torch.empty(d, E, device="cuda").normal_(generator=g)
    ids = torch.stack([torch.arange(T, device="cuda") % E, (torch.arange(T, device="cuda") + 1) % E], 1).to(torch.int32)
    w = torch.empty(T, k, device="cuda").uniform_(0.1, 0.9, generator=g)
    dw = torch.empty(T, k, device="cuda").normal_(generator=g)
    dx, dwg = torch.zeros(T, d, device="cuda"), torch.full((d, E), float("nan"), device="cuda")
    ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    B.moe_gate_topk_bwd(s, x, wg, ids, w, dw, dx, dwg, ws)
    dl = torch.zeros(T, E, device="cuda").scatter_(1, ids.long(), w * (dw - (w * dw).sum(1, keepdim=True)))
    part = lambda t, i: t[i:i + (1 << 22)].double()
    ref = 0.0
    for i in range(0, T, 1 << 22):
        want = part(dl, i) @ wg.double().t()
        assert float((part(dx, i) - want).abs().max()) <= 1e-5 * 32, i   # sums of three products of magnitude up to about 32
        ref = ref + part(x, i).t() @ part(dl, i)
    # fp32 partial sums of 2^18 chunks added one after the other: their roundings, 2^-24 of the running sum each, add up
    # like a random walk to 2^9 * 2^-24 of it
    assert float((dwg.double() - ref).abs().max()) <= 1e-4 * float(ref.abs().max())


# the gate weight's gradient: token chunks of 64 to 512 (one token, a stage, its neighbours, several chunks with a rest), tiles of
# 128 columns and their remainders, 16-expert blocks and 64-expert tiles, and the grouped GEMM (the last two)
@pytest.mark.parametrize("T,d,E,k", [(1, 8, 1, 1), (63, 120, 15, 2), (64, 128, 16, 3), (65, 136, 17, 4), (129, 264, 64, 1),
                                     (700, 1096, 65, 6), (300, 520, 130, 8), (2049, 640, 100, 2), (4097, 136, 200, 4),
                                     (20000, 4096, 8, 2), (131072, 136, 200, 2), (262145, 136, 130, 1)])
def test_gate_weight_gradient_edges(T, d, E, k):
    """Against 64 bits.  The gradient of a logit enters as a pair of bf16 values (2^-17 of it is lost), sums are in fp32:
    1e-5 of the result's 2-norm."""
    g = torch.Generator(device="cuda").manual_seed(T + d + E)
    s = B.Shape(T, d, 8, E, k, torch.bfloat16)
    x = torch.empty(T, d, dtype=torch.bfloat16, device="cuda").normal_(generator=g)
    wg = torch.empty(d, E, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g)
    ids = torch.rand(T, E, device="cuda", generator=g).topk(k, 1).indices.int().contiguous()
    w, dw = torch.softmax(torch.randn(T, k, device="cuda", generator=g), 1), torch.randn(T, k, device="cuda", generator=g)
    dwg = torch.full((d, E), float("nan"), device="cuda")
    ws = torch.full((B.moe_workspace_bytes(s),), 255, dtype=torch.uint8, device="cuda")   # (NaNs in whatever is not written)
    B.moe_gate_topk_bwd(s, x, wg, ids, w, dw, None, dwg, ws)
    dl = w.double() * (dw.double() - (w.double() * dw.double()).sum(1, keepdim=True))
    want = x.double().T @ torch.zeros(T, E, dtype=torch.float64, device="cuda").scatter_(1, ids.long(), dl)
    assert float((dwg.double() - want).norm()) <= 1e-5 * float(want.norm()) + 1e-30
