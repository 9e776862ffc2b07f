"""GPU parity of the token dispatcher (moe_permute_lite, moe_grouped_ffn_fwd_groups) through the C ABI:
integer outputs bit-exact against oracle/lite_oracle.py; the layer output over replica groups bit-identical
to the plain path (replicas share weights) and within the bf16 bar of the CPU oracle."""
import numpy as np
import pytest
import torch

from oracle import lite_oracle as DO
from oracle import oracle as O
from oracle import planner_oracle as PO
from paper_2602_11686_amd import binding as B
from paper_2602_11686_amd import inputs as I
from tests.gpu_common import TOL, host
from tests.helpers import rel_max, rel_max_blocks

pytestmark = pytest.mark.gpu


def i32(a):
    return torch.tensor(np.asarray(a, dtype=np.int32), dtype=torch.int32, device="cuda")


def layout_for(ids, E, N, C, Dn, rank, seed):
    """A layout from the planner oracle for a cluster in which `rank` holds these ids and the other devices
    hold seeded random loads of the same skew."""
    rng = np.random.default_rng(seed)
    mine = np.bincount(ids.reshape(-1), minlength=E)
    R = rng.poisson(np.maximum(mine, 1)[None, :] * rng.uniform(0.5, 1.5, size=(N, 1))).astype(np.int64)
    R[rank] = mine
    A = PO.expert_relocation(PO.replica_allocation(R.tolist(), N, E, C), R.sum(axis=0).tolist(), N, E, C, Dn)
    return DO.dispatch_table(A, N, E, Dn, rank)


def random_ids(seed, T, E, k, skew=1.5):
    rng = np.random.default_rng(seed)
    w = 1.0 / np.arange(1, E + 1) ** skew
    w = w[rng.permutation(E)]
    g = rng.gumbel(size=(T, E)) + np.log(w)[None, :]
    return np.argsort(-g, axis=1)[:, :k].astype(np.int32)


def run_permute_lite(s, G, x, ids, rb, rg):
    ec = torch.empty(s.E, dtype=torch.int32, device="cuda")
    gc = torch.empty(G, dtype=torch.int32, device="cuda")
    go = torch.empty(G + 1, dtype=torch.int32, device="cuda")
    rop = torch.empty(s.R, dtype=torch.int32, device="cuda")
    por = torch.empty(s.R, dtype=torch.int32, device="cuda")
    xp = torch.empty(s.R, s.d, dtype=s.dtype, device="cuda") if x is not None else None
    err = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    B.moe_permute_lite(s, G, x, i32(ids), i32(rb), i32(rg), ec, gc, go, rop, por, xp, err, ws)
    torch.cuda.synchronize()
    return ec, gc, go, rop, por, xp, err


CASES = [  # T, E, k, N, C, D, rank
    (1, 4, 2, 4, 2, 2, 1),
    (300, 8, 2, 8, 2, 4, 5),
    (1000, 8, 2, 32, 2, 8, 9),
    (777, 64, 4, 32, 4, 8, 31),
    (2048, 130, 3, 64, 4, 8, 17),
    (513, 16, 16, 16, 2, 8, 0),
    (4096, 128, 8, 32, 8, 8, 12),
    (8192, 64, 4, 32, 4, 8, 5),      # cfg2's routing shape on a 32-device cluster, G = 128
    (16384, 8, 2, 32, 2, 8, 20),     # cfg3's (Mixtral e8k2, the paper's cluster: 4 nodes of 8, C = 2), G = 64
]


@pytest.mark.parametrize("T,E,k,N,C,Dn,rank", CASES)
def test_permute_lite_matches_the_oracle(T, E, k, N, C, Dn, rank):
    print(f"case T={T} E={E} k={k} N={N} C={C} D={Dn} rank={rank}", flush=True)
    ids = random_ids(T + E, T, E, k)
    G, eog, dog, rb, rg = layout_for(ids, E, N, C, Dn, rank, seed=T)
    assert G <= 256
    d = 64
    s = B.Shape(T, d, 64, E, k, torch.bfloat16)
    x = torch.randn(T, d, device="cuda").bfloat16()
    ec, gc, go, rop, por, xp, err = run_permute_lite(s, G, x, ids, rb, rg)
    r_ec, r_gc, r_go, r_rop, r_por = DO.permute_lite(ids.tolist(), E, G, rb, rg)
    assert int(err[0]) == 0
    assert host(ec).tolist() == r_ec and host(gc).tolist() == r_gc and host(go).tolist() == r_go
    assert host(rop).tolist() == r_rop and host(por).tolist() == r_por
    src = torch.tensor(np.asarray(r_por) // k, device="cuda")
    assert torch.equal(xp.view(torch.int16), x[src].view(torch.int16))          # rows are bitwise copies


def test_without_replication_equals_moe_permute():
    T, E, k, d = 2000, 32, 4, 128
    ids = random_ids(5, T, E, k)
    s = B.Shape(T, d, 64, E, k, torch.bfloat16)
    x = torch.randn(T, d, device="cuda").bfloat16()
    ec, gc, go, rop, por, xp, err = run_permute_lite(s, E, x, ids, list(range(E + 1)), list(range(E)))
    counts = torch.empty(E, dtype=torch.int32, device="cuda"); offsets = torch.empty(E + 1, dtype=torch.int32, device="cuda")
    rop2 = torch.empty_like(rop); por2 = torch.empty_like(por); xp2 = torch.empty_like(xp)
    ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    B.moe_permute(s, x, i32(ids), counts, offsets, rop2, por2, xp2, ws)
    torch.cuda.synchronize()
    assert int(err[0]) == 0 and torch.equal(gc, counts) and torch.equal(go, offsets) and torch.equal(ec, counts)
    assert torch.equal(rop, rop2) and torch.equal(por, por2) and torch.equal(xp.view(torch.int16), xp2.view(torch.int16))


@pytest.mark.parametrize("what", ["no_list", "group_out_of_range", "group_twice", "list_out_of_bounds", "decreasing"])
def test_a_bad_table_is_reported_and_stays_in_bounds(what):
    T, E, k, G = 500, 8, 2, 12
    ids = random_ids(11, T, E, k, skew=0.5)            # every expert has pairs
    rb = list(range(E + 1)); rg = list(range(E))
    if what == "no_list":
        rb = [0, 0] + list(range(1, E)); rg = list(range(E - 1))        # expert 0 has pairs but no replica
    elif what == "group_out_of_range":
        rg[3] = G
    elif what == "group_twice":
        rg[5] = rg[2]
    elif what == "list_out_of_bounds":
        rb[E] = E + 3
    elif what == "decreasing":
        rb[4] = 2
    s = B.Shape(T, 64, 64, E, k, torch.bfloat16)
    ec, gc, go, rop, por, xp, err = run_permute_lite(s, G, None, ids, rb, rg)
    assert int(err[0]) != 0
    counts = np.bincount(ids.reshape(-1), minlength=E)
    assert host(ec).tolist() == counts.tolist()
    assert host(gc).tolist() == [T * k] + [0] * (G - 1) and host(go).tolist() == [0] + [T * k] * G
    x = np.zeros((T, 4), np.float32)
    _, _, r_rop, r_por, _ = O.permute(x, ids, E)  # plain expert order
    assert host(rop).tolist() == r_rop.tolist() and host(por).tolist() == r_por.tolist()


@pytest.mark.parametrize("T,d,f,E,k,N,C,Dn,rank", [(600, 256, 384, 8, 2, 8, 2, 4, 3), (1500, 512, 256, 16, 4, 16, 4, 8, 9),
                          (900, 128, 128, 64, 4, 32, 8, 8, 3)])   # the last one: G = 256 groups, the most the tables hold
def test_layer_over_replica_groups(T, d, f, E, k, N, C, Dn, rank):
    """permute_lite -> grouped FFN over groups -> combine gives the bits of permute -> grouped FFN -> combine,
    and both sit within the bf16 bar of the oracle's layer."""
    print(f"case T={T} d={d} f={f} E={E} k={k}", flush=True)
    rng = np.random.default_rng(T)
    bits = lambda a: I.f32_to_bf16_bits(a.astype(np.float32))
    xb = bits(rng.standard_normal((T, d))); w1b = bits(rng.standard_normal((E, d, f)) * 0.05)
    w3b = bits(rng.standard_normal((E, d, f)) * 0.05); w2b = bits(rng.standard_normal((E, f, d)) * 0.05)
    ids = random_ids(T, T, E, k)
    wts = rng.random((T, k)).astype(np.float32); wts /= wts.sum(1, keepdims=True)
    G, eog, dog, rb, rg = layout_for(ids, E, N, C, Dn, rank, seed=1)
    to = lambda b: torch.tensor(b.view(np.int16), device="cuda").view(torch.bfloat16)
    x, w1, w3, w2 = to(xb), to(w1b), to(w3b), to(w2b)
    s = B.Shape(T, d, f, E, k, torch.bfloat16)
    ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    tw = torch.tensor(wts, device="cuda")
    # plain path
    counts = torch.empty(E, dtype=torch.int32, device="cuda"); offsets = torch.empty(E + 1, dtype=torch.int32, device="cuda")
    rop = torch.empty(s.R, dtype=torch.int32, device="cuda"); por = torch.empty_like(rop)
    xp = torch.empty(s.R, d, dtype=torch.bfloat16, device="cuda"); yp = torch.empty_like(xp); y = torch.empty_like(x)
    B.moe_permute(s, x, i32(ids), counts, offsets, rop, por, xp, ws)
    B.moe_grouped_ffn_fwd(s, xp, offsets, w1, w3, w2, yp, None, None, ws)
    B.moe_unpermute_combine(s, yp, rop, tw, y)
    # lite path
    ec, gc, go, rop_l, por_l, xp_l, err = run_permute_lite(s, G, x, ids, rb, rg)
    yp_l = torch.empty_like(xp); y_l = torch.empty_like(x)
    B.moe_grouped_ffn_fwd_groups(s, G, i32(eog), xp_l, go, w1, w3, w2, yp_l, None, None, ws)
    B.moe_unpermute_combine(s, yp_l, rop_l, tw, y_l)
    torch.cuda.synchronize()
    assert int(err[0]) == 0
    assert torch.equal(y.view(torch.int16), y_l.view(torch.int16))
    assert torch.equal(yp[rop.long()].view(torch.int16), yp_l[rop_l.long()].view(torch.int16))
    # oracle: grouped FFN over the groups with the weights gathered per group, then the combine
    f64 = lambda b: I.bf16_bits_to_f32(b).astype(np.float64)
    r = DO.permute_lite(ids.tolist(), E, G, rb, rg)
    go_ref, rop_ref, por_ref = np.asarray(r[2], np.int32), np.asarray(r[3], np.int32), np.asarray(r[4], np.int32)
    X = f64(xb)
    Xp = X[por_ref // k]
    e = np.asarray(eog)
    Yp = O.ffn_fwd(Xp, go_ref, f64(w1b)[e], f64(w3b)[e], f64(w2b)[e])[0]
    Y = O.unpermute_combine(Yp, rop_ref, wts.astype(np.float64), T)
    assert rel_max(host(yp_l), Yp) <= TOL[torch.bfloat16]
    assert rel_max(host(y_l), Y) <= TOL[torch.bfloat16]


@pytest.mark.parametrize("T,d,f,E,k,N,C,Dn,rank", [(600, 256, 192, 8, 2, 8, 2, 4, 3), (900, 128, 256, 16, 4, 8, 4, 4, 0)])
def test_backward_over_replica_groups(T, d, f, E, k, N, C, Dn, rank):
    """moe_grouped_ffn_bwd_groups: dx_perm per row against the oracle's FFN backward over the groups (weights
    gathered per group), and the per-group weight gradients summed over the groups of an expert against the
    oracle's per-expert gradients of the plain layout (the reshard step sums replica gradients).  Every
    expert's block is compared on its own scale; saved and recomputed activations give the same bits."""
    print(f"case T={T} d={d} f={f} E={E} k={k}", flush=True)
    rng = np.random.default_rng(T + 1)
    bits = lambda a: I.f32_to_bf16_bits(a.astype(np.float32))
    xb = bits(rng.standard_normal((T, d))); w1b = bits(rng.standard_normal((E, d, f)) * 0.05)
    w3b = bits(rng.standard_normal((E, d, f)) * 0.05); w2b = bits(rng.standard_normal((E, f, d)) * 0.05)
    ids = random_ids(T, T, E, k)
    G, eog, dog, rb, rg = layout_for(ids, E, N, C, Dn, rank, seed=2)
    to = lambda b: torch.tensor(b.view(np.int16), device="cuda").view(torch.bfloat16)
    x, w1, w3, w2 = to(xb), to(w1b), to(w3b), to(w2b)
    s = B.Shape(T, d, f, E, k, torch.bfloat16)
    ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    ec, gc, go, rop_l, por_l, xp_l, err = run_permute_lite(s, G, x, ids, rb, rg)
    assert int(err[0]) == 0
    dypb = bits(rng.standard_normal((s.R, d)))
    dyp = to(dypb)
    bf = dict(dtype=torch.bfloat16, device="cuda")
    yp = torch.empty(s.R, d, **bf); a = torch.empty(s.R, f, **bf); b = torch.empty(s.R, f, **bf)
    eog_d = i32(eog)
    B.moe_grouped_ffn_fwd_groups(s, G, eog_d, xp_l, go, w1, w3, w2, yp, a, b, ws)
    outs = []
    for saved in (True, False):
        dxp = torch.full((s.R, d), float("nan"), **bf)
        dw1 = torch.full((G, d, f), float("nan"), **bf); dw3 = torch.full((G, d, f), float("nan"), **bf)
        dw2 = torch.full((G, f, d), float("nan"), **bf)
        B.moe_grouped_ffn_bwd_groups(s, G, eog_d, xp_l, go, w1, w3, w2, a if saved else None, b if saved else None,
                                     dyp, dxp, dw1, dw3, dw2, ws)
        torch.cuda.synchronize()
        outs.append((dxp, dw1, dw3, dw2))
    for p, q in zip(*outs):
        assert torch.equal(p.view(torch.int16), q.view(torch.int16))
    dxp, dw1, dw3, dw2 = outs[0]
    # oracle over the groups: FFN backward with the weights gathered per group
    f64 = lambda v: I.bf16_bits_to_f32(v).astype(np.float64)
    go_ref = host(go).astype(np.int32)
    e = np.asarray(eog)
    Xp = f64(xb)[host(por_l) // k]
    ref_dxp, g1, g3, g2 = O.ffn_bwd(Xp, go_ref, f64(w1b)[e], f64(w3b)[e], f64(w2b)[e], f64(dypb))
    tol = TOL[torch.bfloat16]
    groups = [slice(int(go_ref[g]), int(go_ref[g + 1])) for g in range(G)]
    from tests.helpers import rel_max_blocks
    assert rel_max(host(dxp), ref_dxp) <= tol
    err_b, gi = rel_max_blocks(host(dxp), ref_dxp, groups)
    assert err_b <= tol, ("dXp", "group", gi, err_b)
    for name, got, want in (("dW1", dw1, g1), ("dW3", dw3, g3), ("dW2", dw2, g2)):
        got = host(got)
        assert np.isfinite(got).all(), name
        err_b, gi = rel_max_blocks(got, want, range(G))
        assert err_b <= tol, (name, "group", gi, err_b)
        # summed over the groups of an expert: the expert's gradient in the plain (un-replicated) layout
        summed = np.zeros((E,) + got.shape[1:])
        np.add.at(summed, e, got)
        want_e = np.zeros_like(summed)
        np.add.at(want_e, e, want)
        err_e, ei = rel_max_blocks(summed, want_e, range(E))
        assert err_e <= tol, (name, "expert", ei, err_e)
    for g in np.nonzero(np.diff(go_ref) == 0)[0]:
        assert float(dw1[g].abs().max()) == 0 and float(dw2[g].abs().max()) == 0 and float(dw3[g].abs().max()) == 0


# 17 to 192 rows per group on average and enough column tiles to fill the chip: the instances of the tile kernel that look
# for groups with weights to themselves.  Replicas, an expert of one group, a replica without rows, entries out of range,
# groups of one to three row tiles
@pytest.mark.parametrize("counts,eog", [((64,) * 32, [g % 8 for g in range(32)]),
                                        ((100, 0, 1, 129, 300, 64, 128, 65) * 4, [g // 2 for g in range(32)]),
                                        ((20,) * 30 + (600, 0), [0] * 16 + list(range(14)) + [99, -3]),
                                        ((192,) * 32, list(range(32)))])
def test_few_row_groups_equal_the_plain_path_over_their_weights(counts, eog):
    G, d, f = len(counts), 1280, 1024
    E = 32 if max(eog[:-2]) >= 16 else 16
    g = torch.Generator(device="cuda").manual_seed(sum(counts))
    val = lambda *n, std=1.0: torch.empty(*n, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
    R = sum(counts)
    off = i32(np.concatenate([[0], np.cumsum(counts)]))
    x, dy, w1, w3, w2 = val(R, d), val(R, d), val(E, d, f, std=0.02), val(E, d, f, std=0.02), val(E, f, d, std=0.02)
    at = torch.tensor(eog, device="cuda").clamp(0, E - 1)

    def run(fwd, bwd, shape):
        nan = lambda *n: torch.full(n, float("nan"), dtype=torch.bfloat16, device="cuda")
        y, a, b, dx, g1, g3, g2 = nan(R, d), nan(R, f), nan(R, f), nan(R, d), nan(G, d, f), nan(G, d, f), nan(G, f, d)
        ws = torch.empty(B.moe_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
        fwd(y, a, b, ws)
        bwd(a, b, dx, g1, g3, g2, ws)
        return y, a, b, dx, g1, g3, g2

    s = B.Shape(R, d, f, E, 1, torch.bfloat16)
    got = run(lambda y, a, b, ws: B.moe_grouped_ffn_fwd_groups(s, G, i32(eog), x, off, w1, w3, w2, y, a, b, ws),
              lambda a, b, dx, g1, g3, g2, ws: B.moe_grouped_ffn_bwd_groups(s, G, i32(eog), x, off, w1, w3, w2, a, b, dy, dx, g1,
                                                                            g3, g2, ws), s)
    p = B.Shape(R, d, f, G, 1, torch.bfloat16)
    v1, v3, v2 = w1[at], w3[at], w2[at]
    want = run(lambda y, a, b, ws: B.moe_grouped_ffn_fwd(p, x, off, v1, v3, v2, y, a, b, ws),
               lambda a, b, dx, g1, g3, g2, ws: B.moe_grouped_ffn_bwd(p, x, off, v1, v3, v2, a, b, dy, dx, g1, g3, g2, ws), p)
    for u, v in zip(got, want):
        assert torch.isfinite(u).all() and torch.equal(u, v)


# An expert's rows cut into groups: the rows keep their order and their results must keep their bits, although the mean rows per group
# and the number of tiles, by which the bf16 and fp32 kernels are chosen, are not those of the experts.  Replicas without rows, entries
# out of range (the first below, the last above).  Where the line to the fp32 kernel with a split contraction, counted over groups
# instead of experts, would put the groups on the other side; fp32 tiles of 128x128 (experts) and 64x64 (groups); the fp32 products
# behind dH in one launch (small); on the split kernel by the mean rows alone (at most 16 per expert, 24 experts); bf16 with 64 rows
# per expert and 16 per group, and with contractions that are no multiple of 64
GROUPED = {"f32 W1|W3, dgrad 1": (torch.float32, [16] * 32, [g // 4 for g in range(32)], 8, 512, 1024),
           "f32 W1|W3 the other way": (torch.float32, [16, 0, 41, 8] * 8, [g // 4 for g in range(32)], 8, 128, 192),
           "f32 large": (torch.float32, [128] * 15 + [150], [g // 8 for g in range(16)], 2, 36, 7300),
           "f32 small": (torch.float32, [5, 33, 0, 64, 31, 0, 40, 1], [-3, 0, 1, 1, 2, 3, 3, 99], 4, 100, 68),
           "f32 few rows": (torch.float32, [9, 0, 1, 16, 3, 7] * 8, [g // 2 for g in range(48)], 24, 1028, 776),
           "bf16": (torch.bfloat16, [16] * 31 + [9], [-1] + [g // 4 for g in range(1, 31)] + [8], 8, 512, 768),
           "bf16 remainders": (torch.bfloat16, [30, 0, 33, 1] * 8, [g // 4 for g in range(32)], 8, 520, 776)}


@pytest.mark.parametrize("case", GROUPED)
def test_groups_of_an_experts_rows_give_its_bits(case):
    dt, counts, eog, E, d, f = GROUPED[case]
    print(f"case {case}", flush=True)
    G, R = len(counts), sum(counts)
    at = np.clip(eog, 0, E - 1)
    g_off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    e_off = np.concatenate([[0], np.cumsum(np.bincount(at, weights=counts, minlength=E))]).astype(np.int32)
    assert (np.diff(at) >= 0).all()
    rng = np.random.default_rng(R + d)
    values = lambda *n, std=1.0: torch.from_numpy((rng.standard_normal(n) * std).astype(np.float32)).to(dt)
    data = x, dy, w1, w3, w2 = values(R, d), values(R, d), values(E, d, f, std=0.05), values(E, d, f, std=0.05), values(E, f, d, std=0.05)
    x, dy, w1, w3, w2 = (v.cuda() for v in data)
    s = B.Shape(R, d, f, E, 1, dt)
    ws = torch.empty(B.moe_workspace_bytes(s), dtype=torch.uint8, device="cuda")
    nan = lambda *n: torch.full(n, float("nan"), dtype=dt, device="cuda")
    y, a, b, dx, g1, g3, g2 = nan(R, d), nan(R, f), nan(R, f), nan(R, d), nan(E, d, f), nan(E, d, f), nan(E, f, d)
    B.moe_grouped_ffn_fwd(s, x, i32(e_off), w1, w3, w2, y, a, b, ws)
    B.moe_grouped_ffn_bwd(s, x, i32(e_off), w1, w3, w2, a, b, dy, dx, g1, g3, g2, ws)
    yg, ag, bg, dxg, g1, g3, g2 = nan(R, d), nan(R, f), nan(R, f), nan(R, d), nan(G, d, f), nan(G, d, f), nan(G, f, d)
    B.moe_grouped_ffn_fwd_groups(s, G, i32(eog), x, i32(g_off), w1, w3, w2, yg, ag, bg, ws)
    B.moe_grouped_ffn_bwd_groups(s, G, i32(eog), x, i32(g_off), w1, w3, w2, ag, bg, dy, dxg, g1, g3, g2, ws)
    torch.cuda.synchronize()
    for name, u, v in (("A", a, ag), ("B", b, bg), ("Yp", y, yg), ("dXp", dx, dxg)):
        assert torch.isfinite(u).all() and torch.equal(u, v), name
    # the gradients of the groups, against the oracle over the gathered weights
    x, dy, w1, w3, w2 = (v.double().numpy() for v in data)
    ref_dx, r1, r3, r2 = O.ffn_bwd(x, g_off, w1[at], w3[at], w2[at], dy)
    assert rel_max(host(dxg), ref_dx) <= TOL[dt]
    for name, got, want in (("dW1", g1, r1), ("dW3", g3, r3), ("dW2", g2, r2)):
        got = host(got)
        assert np.isfinite(got).all(), name
        err, g = rel_max_blocks(got, want, range(G))
        assert err <= TOL[dt], (name, "group", g, err)
