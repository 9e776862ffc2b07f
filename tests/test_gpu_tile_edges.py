"""The expert FFN calls at the sizes where a tile, a remainder or a dispatch rule can go wrong, against the oracle.

Tolerances (largest difference over the largest reference value, per tensor and per expert): bf16 as in the other
stage tests; fp32 2^-24 per rounded sum times the longest contraction here (4096 terms: dX sums two segments of 2048;
worst case 2.4e-4) is covered by their 1e-4 because the errors of a sum partly cancel.
"""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2602_11686_amd import binding as B
from paper_2602_11686_amd import inputs as I
from paper_2602_11686_amd.layer import MoeLayerBuffers
from gpu_common import TOL, host
from helpers import rel_max, rel_max_blocks, row_blocks

pytestmark = pytest.mark.gpu


def check_ffn(counts, d, f, dtype, seed, backward=True, wstd=0.05):
    rng = np.random.default_rng(seed)
    counts = np.array(counts, np.int32)
    E, R = len(counts), int(counts.sum())
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    f32 = dtype == torch.float32

    def values(*shape, std=1.0):
        a = (rng.standard_normal(shape) * std).astype(np.float32)
        if f32:
            return torch.from_numpy(a).cuda(), a.astype(np.float64)
        b = I.f32_to_bf16_bits(a)
        return torch.from_numpy(b.view(np.int16)).cuda().view(torch.bfloat16), I.widen(b, np.float64)

    (xp, xp_o), (dyp, dyp_o) = values(R, d), values(R, d)
    (w1, w1_o), (w3, w3_o), (w2, w2_o) = (values(*n, std=wstd) for n in ((E, d, f), (E, d, f), (E, f, d)))
    yp, A, Bm, H = O.ffn_fwd(xp_o, offsets, w1_o, w3_o, w2_o)
    s = B.Shape(R, d, f, E, 1, dtype)     # T*k = R with k = 1: the shape only sizes the buffers of these calls
    buf = MoeLayerBuffers(s, backward=True)
    off = torch.from_numpy(offsets).cuda()
    rows, tol = row_blocks(offsets), TOL[dtype]

    def check(what, triples):
        torch.cuda.synchronize()
        for name, got, want, blocks in triples:
            got = host(got)
            assert np.isfinite(got).all(), (what, name)
            assert rel_max(got, want) <= tol, (what, name)
            err, e = rel_max_blocks(got, want, blocks)
            assert err <= tol, (what, name, "expert", e, "rows", int(counts[e]), err)

    for t in (buf.y_perm, buf.a_save, buf.b_save, buf.dx_perm, buf.dw1, buf.dw3, buf.dw2):
        t.fill_(float("nan"))
    B.moe_grouped_ffn_fwd(s, xp, off, w1, w3, w2, buf.y_perm, None, None, buf.ws)
    check("inference", [("Yp", buf.y_perm, yp, rows)])
    B.moe_grouped_ffn_fwd(s, xp, off, w1, w3, w2, buf.y_perm, buf.a_save, buf.b_save, buf.ws)
    check("forward", [("Yp", buf.y_perm, yp, rows), ("A", buf.a_save, A, rows), ("B", buf.b_save, Bm, rows)])
    if not backward:
        return
    ref = O.ffn_bwd(xp_o, offsets, w1_o, w3_o, w2_o, dyp_o)
    grads = lambda: [("dXp", buf.dx_perm, ref[0], rows), ("dW1", buf.dw1, ref[1], range(E)),
                     ("dW3", buf.dw3, ref[2], range(E)), ("dW2", buf.dw2, ref[3], range(E))]
    for a, b in ((buf.a_save, buf.b_save), (None, None)):
        B.moe_grouped_ffn_bwd(s, xp, off, w1, w3, w2, a, b, dyp, buf.dx_perm, buf.dw1, buf.dw3, buf.dw2, buf.ws)
        check("backward", grads())
    h = torch.full_like(buf.a_save, float("nan"))
    B.moe_grouped_ffn_fwd_products(s, xp, off, w1, w3, w2, buf.y_perm, h, buf.a_save, buf.b_save)
    B.moe_grouped_ffn_bwd_products(s, xp, off, w1, w3, w2, h, buf.a_save, buf.b_save, dyp, buf.dx_perm, buf.dw1,
                                   buf.dw3, buf.dw2, buf.ws)
    check("products", [("H", h, H, rows)] + grads())
    for e in np.nonzero(counts == 0)[0]:
        assert not buf.dw1[e].any() and not buf.dw3[e].any() and not buf.dw2[e].any()


# fp32, 32x32 and 64x64 tiles (too few for 128x128 ones in every product): remainders of rows, columns and k-stages
@pytest.mark.parametrize("counts,d,f", [((1, 0, 63, 64, 65, 130), 68, 36), ((5, 17), 4, 132), ((0, 129, 300), 64, 16),
                                        ((1200, 127, 0, 1), 2048, 260), ((700, 900), 260, 2048)])
def test_ffn_f32(counts, d, f):
    check_ffn(counts, d, f, torch.float32, 7 * d + f)


# fp32, 32-wide k-stages: none to five of them in either contraction, with every kind of remainder
@pytest.mark.parametrize("counts,d,f", [((28, 32, 36, 0), 32, 64), ((64, 68, 96, 1), 96, 28), ((4, 31, 33, 160), 100, 128),
                                        ((130, 3), 36, 160)])
def test_ffn_f32_stages(counts, d, f):
    check_ffn(counts, d, f, torch.float32, 5 * d + f)


# fp32, 32x32 tiles with the contraction split over four wavefronts: tiles, columns and slabs of 32 with remainders; fewer slabs
# than wavefronts, one more than they can hold in their rings, segments that begin in the middle of the four; few rows per expert
# with many tiles, and with contractions on the two sides of 512; two matrices with a long contraction and tiles that have no rows, and
# with rows in all.  By product over ragged rows (W1|W3, W2, dgrad 1, dX) which are split (s), and whether the three products behind dH
# go into one launch (1), the gradients are split alone (s) or not (-).
@pytest.mark.parametrize("split,counts,d,f", [("ssss1", (31, 0, 32, 33, 1), 36, 68), ("ssss1", (2, 5), 4, 160), ("ssss1", (65, 0, 127), 132, 292),
                                              ("ssss1", (300, 4), 100, 36), ("ssss-", (9, 0, 16, 1, 40, 3) * 4, 1028, 776),
                                              ("-----", (65, 130, 0, 63, 1, 300), 836, 1092), ("-s-s-", (9, 0, 16, 1, 40, 3) * 8, 508, 512),
                                              ("---s-", (9, 0, 16, 1, 40, 3) * 8, 508, 508), ("s-s--", (9, 0, 16, 1, 40, 3) * 8, 512, 252),
                                              ("s-s--", (70, 0, 30, 29), 2048, 1380), ("--s--", (66, 400, 500, 34), 2048, 508)])
def test_ffn_f32_split(split, counts, d, f):
    up = lambda n, m: -(-n // m)
    E, R = len(counts), sum(counts)
    rows, few = up(R, 64) + E, lambda k: R <= 16 * E and k >= 512
    dual = rows * up(f, 32) <= 128 or (d >= 2048 and rows * up(f, 32) <= 320 and up(R, 64) * up(f, 32) <= 192)
    over_rows = [few(d) or dual, few(f) or rows * up(d, 64) <= 192, few(d) or rows * up(f, 64) <= 192, few(2 * f) or rows * up(d, 64) <= 192]
    grads = [E * up(f, 64) * up(d, 64) <= 128, E * up(d, 64) * up(f, 32) <= 128]
    assert "".join("s" if p else "-" for p in over_rows) == split[:4]
    assert ("1" if all(grads + over_rows[3:]) else "s" if all(grads) else "-" if not any(grads) else "?") == split[4]
    check_ffn(counts, d, f, torch.float32, 3 * d + f)


# fp32, 128x128 tiles: enough of them, and of rows per expert, in the named products (an upper bound with ragged rows, as the
# dispatch counts them); remainders of rows, columns and k-stages
@pytest.mark.parametrize("products,counts,d,f", [("dW1", (0, 1, 127, 128, 129, 300, 17, 64) * 25, 260, 264),
                                                 ("dW1 dW2", (0, 1, 127, 128, 129, 300, 17, 64) * 25, 260, 388),
                                                 ("A", (0, 1, 127, 128, 129, 3000, 2500, 2400), 36, 1868),
                                                 ("Yp", (0, 1, 127, 128, 129, 3000, 2500, 2400), 7300, 36),
                                                 ("Yp", (1030, 1100, 1000, 1024), 14980, 4)])
def test_ffn_f32_large_tiles(products, counts, d, f):
    up = lambda n, m: -(-n // m)
    E, R = len(counts), sum(counts)
    rows = up(R, 128) + E
    large = {"A": up(f, 64) * rows >= 2048 and R >= 512 * E, "Yp": up(d, 128) * rows >= 4096 and R >= 1024 * E,
             "dW2": up(d, 128) * up(f, 128) * E >= 2048, "dW1": up(f, 64) * up(d, 128) * E >= 2048}
    assert {p for p in large if large[p]} == set(products.split())
    check_ffn(counts, d, f, torch.float32, 3)


# bf16 leading dimensions beyond the 32-bit offsets of the tile kernels: the plain 128x128x64 kernel
@pytest.mark.parametrize("counts,d,f,wstd", [((3, 2), 1 << 21, 8, 7e-4), ((5,), 8, 1 << 21, 0.05)])
def test_ffn_bf16_huge_leading_dimension(counts, d, f, wstd):
    check_ffn(counts, d, f, torch.bfloat16, 23, wstd=wstd)


# bf16 contractions that end inside a 64-wide stage: one piece, one piece short of a stage, several stages and a rest
@pytest.mark.parametrize("counts,d,f", [((3, 0, 130), 8, 8), ((257, 64, 1), 56, 72), ((128, 300, 2), 200, 328),
                                        ((520, 31), 264, 1096)])
def test_ffn_bf16_k_remainder(counts, d, f):
    check_ffn(counts, d, f, torch.bfloat16, 11 * d + f)


# 256-row tiles computed in quadrants: one to six k-stages, tiles of at most 128 rows (with and without rows in the second
# 64) among full ones, several tiles per workgroup, a last round cut in two, a remainder of K
# (the weight gradients too, from a mean of 80 rows on: experts of no rows, one, a stage, a stage and one; tiles of at most 128
# of their rows; none to three tiles per workgroup from the queues)
@pytest.mark.parametrize("counts,d,f", [((0, 300, 1, 63, 64, 65, 0), 136, 72), ((0, 400, 0, 160), 64, 520), ((81, 79), 384, 640),
                                        # 17 to 192 rows, enough column tiles to fill the chip: non-temporal weights and outputs
                                        ((18,) * 30 + (257, 0), 1024, 1088), ((64, 1, 129) * 12, 768, 1024),
                                        ((400, 0, 30, 200, 100, 129, 1, 90) * 8, 520, 1032), ((300, 1, 0, 128, 129), 64, 64), ((257, 200, 64), 128, 192), ((700, 0, 513), 320, 256),
                                        ((65,) * 30 + (300,) * 10, 1024, 1408), ((2000, 130, 384), 2048, 1032)])
def test_ffn_quadrants(counts, d, f):
    check_ffn(counts, d, f, torch.bfloat16, 19 * d + f)


# d = 64: stages of the whole contraction, so that requests run two tiles ahead; d = 8: a remainder of K
@pytest.mark.parametrize("d", [64, 8])
def test_ffn_quadrants_long_tile_list(d):
    """772 tiles for each workgroup in the first product, which keeps a ring of 512 and refills either half once.  One rounding
    to bf16 (2^-9 of the value) plus fp32 sums (2^-24 of their terms' absolute values each, partly cancelling: 1e-5 of
    them covers 168) of 64 or 8 and of 65528 terms; |silu'| is at most 1.1."""
    E, f, few, big = 256, 65528, 18, 130 * 256 + 5
    counts = [few] * E
    counts[100] = big
    R = sum(counts)
    # the quadrant kernel, by the rules of the dispatch: enough rows, offsets in 32 bits; and its tiles
    assert R > 64 * E and f * f < 1 << 32 and R * f < 1 << 32
    assert sum(-(-c // 256) for c in counts) * -(-f // 128) // 256 > 768
    g = torch.Generator(device="cuda").manual_seed(2)
    off = torch.tensor([0] + np.cumsum(counts).tolist(), dtype=torch.int32, device="cuda")
    val = lambda *n, std=1.0: torch.empty(*n, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    x, w1, w3, w2 = val(R, d), val(E, d, f, std=0.2), val(E, d, f, std=0.2), val(E, f, d)
    s = B.Shape(R, d, f, E, 1, torch.bfloat16)
    y = torch.full((R, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    h, p, q = (torch.full((R, f), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(3))
    B.moe_grouped_ffn_fwd_products(s, x, off, w1, w3, w2, y, h, p, q)
    first = np.concatenate([[0], np.cumsum(counts)])
    for e in range(E):
        a1, a3, a2 = w1[e].double(), w3[e].double(), w2[e].double()
        for b in range(first[e], first[e + 1], 2048):
            r = slice(b, min(b + 2048, first[e + 1]))
            xr, hr = x[r].double(), h[r].double()
            a, c = xr @ a1, xr @ a3
            ta, tc = (xr.abs() @ a1.abs()) * 1e-5, (xr.abs() @ a3.abs()) * 1e-5
            sa = torch.nn.functional.silu(a)
            assert bool(((q[r].double() - sa).abs() <= sa.abs() * 2.0**-8 + 1.1 * ta).all()), (e, b)
            assert bool(((hr - sa * c).abs() <= (sa * c).abs() * 2.0**-8 + 1.1 * ta * c.abs() + tc * sa.abs()).all()), (e, b)
            want, terms = hr @ a2, hr.abs() @ a2.abs()
            assert bool(((y[r].double() - want).abs() <= want.abs() * 2.0**-8 + terms * 1e-5).all()), (e, b)
    assert bool(torch.isfinite(p).all())


# few rows per expert: 64-row tiles (mean at most 32) and 128-row ones (mean 33 .. 64, with and without enough column
# tiles for the wide kernel), 16-row blocks, tails, an expert of several tiles, one to five k-stages and a remainder
@pytest.mark.parametrize("counts,d,f", [((1, 0, 0, 2), 64, 64), ((15, 16, 17, 1, 0, 33, 64, 65), 128, 192),
                                        ((0, 0, 0, 129), 200, 72), ((3,) * 7 + (0, 90), 320, 264),
                                        ((128, 1, 63), 72, 136), ((40, 129, 0, 60), 264, 1096),
                                        ((60,) * 40, 512, 1024), ((20,) * 30 + (300, 0), 1024, 520)])
def test_ffn_few_rows(counts, d, f):
    check_ffn(counts, d, f, torch.bfloat16, 13 * d + f)


# more than 2048 rows per expert on average: the weight gradients go through the instances with plain stores
@pytest.mark.parametrize("counts,d,f", [((6200, 0, 1), 136, 72), ((4100, 300), 264, 520)])
def test_ffn_many_rows(counts, d, f):
    check_ffn(counts, d, f, torch.bfloat16, 17 * d + f)


def test_ffn_f32_more_tiles_than_a_grid_dimension():
    """256 experts of 4 x 2^22: 16.8 million tiles in the first product.  w1, w3 and w2 share 17 GB.  fp32 sums of 2^22
    terms: 2^-24 of the sum of absolute values per addition, which partly cancel; 1e-4 of it is 1678 of them."""
    E, d, f, experts = 256, 4, 1 << 22, (3, 137, 255)
    w = torch.empty(E, d, f, device="cuda").normal_(0.0, 0.5, generator=torch.Generator(device="cuda").manual_seed(1))
    x = torch.tensor([[0.5, -1.0, 2.0, 0.25], [1.5, 0.75, -0.5, 1.0], [-0.25, 1.0, 1.0, -2.0]], device="cuda")
    offsets = torch.tensor([sum(e < i for e in experts) for i in range(E + 1)], dtype=torch.int32, device="cuda")
    s = B.Shape(3, d, f, E, 1, torch.float32)
    y = torch.full((3, d), float("nan"), device="cuda")
    ws = torch.full((3 * f,), float("nan"), device="cuda").view(torch.uint8)
    B.moe_grouped_ffn_fwd(s, x, offsets, w, w, w.view(E, f, d), y, None, None, ws)
    for r, e in enumerate(experts):
        a = x[r].double() @ w[e].double()
        h = torch.nn.functional.silu(a) * a
        w2 = w.view(E, f, d)[e].double()
        assert float(((y[r].double() - h @ w2).abs() / (h.abs() @ w2.abs())).max()) <= 1e-4, e
