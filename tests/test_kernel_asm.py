"""Host-side check of the generated code of the grouped-GEMM kernels fed by LDS DMA (no GPU needed).

The kernels order their LDS DMA loads with hand-placed ``s_waitcnt vmcnt(N)`` in inline assembly, which the
compiler does not see.  If the compiler believes that an ordinary global load is still pending when the
main loop starts (an epilogue load that some path leaves unconsumed, say), it adds waits of its own inside
the loop; they wait for the DMA loads too and cost 15-20 % of the kernel, silently.  So: compile the
kernels to assembly and look at every basic block of the main loops.
"""
import os
import re
import shutil
import subprocess

import pytest

from paper_2602_11686_amd import build as B

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
pytestmark = pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not installed")


@pytest.fixture(scope="module")
def ffn_asm(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "moe_ffn.s"
    cmd = [HIPCC, *B.FLAGS, "-S", "--cuda-device-only", os.path.join(B.CSRC, "moe_ffn.hip"), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return out.read_text()


def kernels(asm, which):
    """{mangled kernel name: [(block label, [instructions])]} for the instances of a kernel."""
    out, kern, label, cur = {}, None, None, []
    for line in asm.split("\n"):
        m = re.match(r"^(_ZN3moe\d+%s\w+):" % which, line)
        if m:
            kern, label, cur = m.group(1), "entry", []
            out[kern] = [(label, cur)]
            continue
        if kern is None:
            continue
        if re.match(r"^\s*\.(size|end_amdhsa_kernel|section)", line) or re.match(r"^_Z\w+:", line):
            kern = None
            continue
        m = re.match(r"^(\.LBB\d+_\d+):", line)
        if m:
            label, cur = m.group(1), []
            out[kern].append((label, cur))
            continue
        t = line.strip()
        if t and not t.startswith(";") and not t.startswith("."):
            cur.append(t)
    return out


def test_main_loops_hold_only_the_hand_placed_vmcnt_waits(ffn_asm):
    ks = kernels(ffn_asm, "gg256_kernel")
    assert len(ks) == 4, sorted(ks)   # the gradients of few rows, the gate's two products: what is launched
    seen_loops = 0
    for name, blocks in ks.items():
        for label, ins in blocks:
            mfma = sum(i.startswith("v_mfma") for i in ins)
            if mfma < 8 or not any("s_barrier" in i for i in ins):
                continue  # not a main-loop block (a stage = MFMAs around one barrier)
            seen_loops += 1
            waits = [(n, int(re.search(r"vmcnt\((\d+)\)", i).group(1))) for n, i in enumerate(ins)
                     if i.startswith("s_waitcnt") and "vmcnt" in i]
            # the one wait of a stage sits right in front of its barrier: the next stage has landed, and since
            # the stage after it is requested only behind the barrier, nothing else is in flight
            assert [w for _, w in waits] == [0], f"{name} {label}: vmcnt waits {waits} inside a main-loop stage"
            bar = next(n for n, i in enumerate(ins) if "s_barrier" in i)
            between = [i for i in ins[waits[0][0] + 1:bar] if i.startswith(("ds_read", "global_load", "buffer_load"))]
            assert 0 < bar - waits[0][0] and not between, f"{name} {label}: the wait is not the one in front of the barrier"
    assert seen_loops >= len(ks)


def test_few_rows_pipeline_holds_only_the_hand_placed_vmcnt_waits(ffn_asm):
    """gg_few_rows_kernel keeps S-2 stages of DMA in flight behind ``vmcnt((S-2)*(CA+CB))``: between its first DMA load
    and its last MFMA the compiler adds no vmcnt wait, the written ones are that and 0, and what follows each of them
    before any DMA request or MFMA is the stage's barrier.  (Two loops: plain and non-temporal weight requests.)"""
    found = 0
    for m in re.finditer(r"^_ZN3moe18gg_few_rows_kernelILi[01]ELb[01]ELi\dELi(\d+)ELi(\d)ELi(\d)E\w+:(.*?)\n\s*s_endpgm",
                         ffn_asm, re.S | re.M):
        bm, nb, stages = (int(m.group(i)) for i in (1, 2, 3))
        lines = [l.strip() for l in m.group(4).split("\n")]
        dma = [n for n, l in enumerate(lines) if l.startswith("global_load_lds")]
        mfma = [n for n, l in enumerate(lines) if l.startswith("v_mfma")]
        assert dma and mfma, m.group(0)[:80]
        by_hand, waits = False, []
        for n in range(dma[0], mfma[-1]):
            if lines[n].startswith(";;#ASM"):
                by_hand = lines[n].startswith(";;#ASMSTART")
            elif lines[n].startswith("s_waitcnt") and "vmcnt" in lines[n]:
                assert by_hand, (m.group(0)[:80], n, lines[n])
                waits.append((n, int(re.search(r"vmcnt\((\d+)\)", lines[n]).group(1))))
        assert sorted({w for _, w in waits}) == sorted({0, (stages - 2) * (bm // 32 + 2 * nb)}), (m.group(0)[:80], waits)
        marks = [(n, l) for n, l in enumerate(lines) if l.startswith(("s_barrier", "v_mfma", "global_load_lds"))]
        for w, _ in waits:
            assert next(l for n, l in marks if n > w).startswith("s_barrier"), (m.group(0)[:80], w)
        assert len([n for n, l in marks if l.startswith("s_barrier")]) == 2, m.group(0)[:80]
        found += 1
    assert found >= 8   # the instances that are launched: 2 forward 1, 2 forward 2, 2 of each of three dgrad epilogues


def test_look_ahead_draw_is_first_read_behind_a_full_wait(ffn_asm):
    """The queue draw for the next tile is a returning atomic issued from inline assembly; its result arrives
    asynchronously.  The only reader of the destination register must be the LDS store that publishes it, and
    that store must follow an s_waitcnt vmcnt(0) in its own straight-line code."""
    found = 0
    # (template arguments AT, BT, DUAL, EPI, RAGK, ...: the ones with ragged K)
    for m in re.finditer(r"^(_ZN3moe12gg256_kernelILi\dELi\dELb[01]ELi\dELb1E\w+):(.*?)\n\s*s_endpgm", ffn_asm, re.S | re.M):
        lines = [l.strip() for l in m.group(2).split("\n")]
        lines = [l for l in lines if l and not l.startswith(";") and (not l.startswith(".") or l.startswith(".LBB"))]
        for n, l in enumerate(lines):
            a = re.match(r"global_atomic_add (v\d+), v\[\d+:\d+\], v\d+, off sc0", l)
            if not a:
                continue
            found += 1
            reg = a.group(1)
            word = re.compile(r"\b%s\b" % reg)
            readers = []
            for k in range(n + 1, len(lines)):
                x = lines[k]
                if not word.search(x):
                    continue
                if re.match(r"\S+ %s\b" % reg, x) and not x.startswith(("ds_write", "global_store", "buffer_store")):
                    break          # the register gets a new value: the draw's life ends here
                readers.append((k, x))
            assert readers, (m.group(1), "the draw is never read")
            for k, x in readers:
                assert re.match(r"ds_write_b32 v\d+, %s$" % reg, x), (m.group(1), x)
                back = lines[max(0, k - 40):k]
                labels = [i for i, y in enumerate(back) if y.startswith(".LBB")]
                straight = back[labels[-1] + 1:] if labels else back
                # the wait may sit in the block in front of the predicated store: look through one label
                window = straight if any("vmcnt(0)" in y for y in straight) else back
                assert any(y.startswith("s_waitcnt") and "vmcnt(0)" in y for y in window), (m.group(1), x)
    assert found >= 2   # the two weight-gradient products draw their tiles


def test_kernels_do_not_spill(ffn_asm):
    for m in re.finditer(r"\.amdhsa_kernel (_ZN3moe\d+gg(?:256|_few_rows)_kernel\w+)(.*?)\.end_amdhsa_kernel", ffn_asm, re.S):
        body = m.group(2)
        scratch = re.search(r"\.amdhsa_private_segment_fixed_size (\d+)", body)
        assert scratch and int(scratch.group(1)) == 0, (m.group(1), scratch and scratch.group(1))
        vgpr = re.search(r"\.amdhsa_next_free_vgpr (\d+)", body)
        assert vgpr and int(vgpr.group(1)) <= 256, (m.group(1), vgpr and vgpr.group(1))


def stage_loop(lines, mfmas):
    """First and last line of the innermost loop with so many MFMAs."""
    label = {m.group(1): n for n, l in enumerate(lines) if (m := re.match(r"(\.LBB\d+_\d+):", l))}
    edges = [(label[m.group(1)], n) for n, l in enumerate(lines) if (m := re.match(r"s_c?branch\w*\s+(\.LBB\d+_\d+)", l))]
    count = lambda h, n: sum(l.startswith("v_mfma") for l in lines[h:n])
    head, last = max((h, n) for h, n in edges if h < n and count(h, n) == mfmas)
    while True:   # what jumps back into it from behind, and what it jumps back to, belongs to it
        h = min([h for h, n in edges if h < head <= n <= last] + [head])
        n = max([n for h, n in edges if head <= h <= last < n] + [last])
        if (h, n) == (head, last):
            break
        head, last = h, n
    assert count(head, last) == mfmas
    return head, last


def test_quadrant_pipeline_holds_only_the_hand_placed_vmcnt_waits(ffn_asm):
    """gg_quad_kernel counts its DMA loads across stages and tiles.  The loop of tiles of more than 128 rows waits in a stage for
    all but 8 of them and then for all but 6, the loop of the others for all but 4 and then 6; each wait stands in front of
    its barrier with nothing read or requested between, and no other vmcnt wait is in the loops, whether in
    a block with MFMAs or not; nothing spills."""
    found = re.findall(r"^(_ZN3moe\d+gg_quad_kernel\w+):(.*?)^\.Lfunc_end", ffn_asm, re.S | re.M)
    assert len(found) == 19, [name for name, _ in found]
    for name, text in found:
        lines = [l.strip() for l in text.split("\n")]
        for mfmas, counted in ((64, [8, 6]), (32, [4, 6])):
            head, last = stage_loop(lines, mfmas)
            by_hand, waits = False, []
            for n in range(head, last):
                l = lines[n]
                if l.startswith(";;#ASM"):
                    by_hand = l.startswith(";;#ASMSTART")
                elif l.startswith("s_waitcnt") and "vmcnt" in l:
                    assert by_hand, (name, mfmas, l)
                    waits.append(int(re.search(r"vmcnt\((\d+)\)", l).group(1)))
                    after = next(x for x in lines[n + 1:] if x.startswith(("s_barrier", "global_", "ds_", "s_cbranch")))
                    assert after.startswith("s_barrier"), (name, mfmas, after)
            assert waits == counted, (name, mfmas, waits)
            assert sum(l.startswith("s_barrier") for l in lines[head:last]) == 2, (name, mfmas)
    for m in re.finditer(r"\.amdhsa_kernel (_ZN3moe\d+gg_quad_kernel\w+)(.*?)\.end_amdhsa_kernel", ffn_asm, re.S):
        assert re.search(r"\.amdhsa_private_segment_fixed_size 0\b", m.group(2)), m.group(1)


def test_quadrant_kernel_counts_the_groups_that_share_weights(ffn_asm):
    """The instances with ragged M that request a single tile's weights non-temporally count in LDS how many groups with rows
    have each expert: replicas read the same weights.  The others have no use for the counts."""
    counting = {}
    for name, blocks in kernels(ffn_asm, "gg_quad_kernel").items():
        _, ragk, stream = re.search(r"ELb([01])ELb([01])ELb([01])EEE", name).groups()
        counts = any(i.startswith("ds_add_") for _, ins in blocks for i in ins)
        assert counts == (ragk == "0" and stream == "1"), name
        counting[name] = counts
    assert sum(counting.values()) == 5, counting   # two forward and three backward products


def test_which_outputs_the_quadrant_kernel_stores_non_temporally(ffn_asm):
    """All of the instances made for that (few rows per expert; the gradients) but the derivative epilogues, and no others."""
    for name, blocks in kernels(ffn_asm, "gg_quad_kernel").items():
        epilogue, stream = re.search(r"kernelILi\dELb[01]ELi(\d)ELb[01]ELb[01]ELb([01])EEE", name).groups()
        nt = {" nt" in i for _, ins in blocks for i in ins if i.startswith("global_store_dwordx4")}
        assert nt == {stream == "1" and epilogue not in "36"}, (name, nt)   # 3, 6: EPI_DH, EPI_DHP


def test_large_fp32_tiles_are_built_for_the_products_that_take_them(ffn_asm):
    """Two forward products and two gradients; the accumulators of a 128x128 tile fit the registers."""
    found = re.findall(r"\.amdhsa_kernel (_ZN3moe\d+gg_f32_large_kernel\w+)(.*?)\.end_amdhsa_kernel", ffn_asm, re.S)
    assert len(found) == 4, [name for name, _ in found]
    for name, body in found:
        assert re.search(r"\.amdhsa_private_segment_fixed_size 0\b", body), name


def test_quadrant_kernel_meets_no_barrier_twice_in_a_row(ffn_asm):
    for name, blocks in kernels(ffn_asm, "gg_quad_kernel").items():
        for label, ins in blocks:
            seen = False   # a barrier, and nothing after it that another wavefront could see
            for i in ins:
                assert not (seen and i.startswith("s_barrier")), (name, label)
                if i.startswith("s_barrier"):
                    seen = True
                elif i.startswith(("ds_", "global_", "v_mfma", "s_cbranch", "s_branch")):
                    seen = False


def hand_placed_waits(lines, first, last):
    """[(line, count)] of the vmcnt waits in between, all of which must be written in inline assembly."""
    by_hand, waits = False, []
    for n in range(first, last):
        if lines[n].startswith(";;#ASM"):
            by_hand = lines[n].startswith(";;#ASMSTART")
        elif lines[n].startswith("s_waitcnt") and "vmcnt" in lines[n]:
            assert by_hand, (n, lines[n])
            waits.append((n, int(re.search(r"vmcnt\((\d+)\)", lines[n]).group(1))))
    return waits


def test_fp32_ring_holds_only_the_hand_placed_vmcnt_waits(ffn_asm):
    """gg_f32_kernel: one stage of DMA (four requests) stays in flight behind a wait, each wait stands in front of the stage's barrier.  The
    forward products compute one 32x32 block per wavefront, the others 2x2 blocks of 16x16."""
    found = re.findall(r"^(_ZN3moe13gg_f32_kernelILi([01])ELi([01])\w+):(.*?)^\.Lfunc_end", ffn_asm, re.S | re.M)
    assert len(found) == 7, [f[0] for f in found]
    for name, at, bt, text in found:
        lines = [l.strip() for l in text.split("\n")]
        mfma = [l.split()[0] for l in lines if l.startswith("v_mfma")]
        assert mfma == (["v_mfma_f32_32x32x2_f32"] * 16 if at + bt == "00" else ["v_mfma_f32_16x16x4_f32"] * 32), name
        waits = hand_placed_waits(lines, *stage_loop(lines, len(mfma)))
        assert sorted(w for _, w in waits) == [0, 4], (name, waits)
        for w, _ in waits:
            assert next(l for l in lines[w + 1:] if l.startswith(("s_barrier", "v_mfma", "global_load_lds", "ds_read"))).startswith("s_barrier"), name


def test_fp32_split_rings_hold_only_the_hand_placed_waits(ffn_asm):
    """gg_f32_split_kernel and the three products of gg_f32_split_bwd_kernel: a wavefront's ring has no barrier, so what orders it are
    its waits.  One slab of DMA (eight requests) stays in flight behind ``vmcnt(8)``, the last slab is waited for with 0, the compiler
    adds no vmcnt wait, and a slab is requested anew only behind an ``lgkmcnt(0)`` that follows its last LDS read."""
    tiles = {}
    for m in re.finditer(r"^(_ZN3moe\d+gg_f32_split(?:_bwd)?_kernel\w+):(.*?)^\.Lfunc_end", ffn_asm, re.S | re.M):
        name, lines = m.group(1), [l.strip() for l in m.group(2).split("\n")]
        at, tiles[name] = 0, 0
        while any(l.startswith("global_load_lds") for l in lines[at:]):
            first = next(n for n in range(at, len(lines)) if lines[n].startswith("global_load_lds"))
            end = next(n for n in range(first, len(lines)) if lines[n].startswith("ds_write"))   # the four sums
            mfma = [n for n in range(first, end) if lines[n].startswith("v_mfma")]
            assert len(mfma) == 32, (name, len(mfma))
            assert sorted(w for _, w in hand_placed_waits(lines, first, mfma[-1])) == [0, 8], name
            reads = [n for n in range(first, mfma[-1]) if lines[n].startswith("ds_read")]
            refill = [n for n in range(reads[0], mfma[-1]) if lines[n].startswith("global_load_lds")]
            assert len(refill) == 8 and refill[0] > reads[-1], name
            assert any(l.startswith("s_waitcnt") and "lgkmcnt(0)" in l for l in lines[reads[-1]:refill[0]]), name
            assert not any(l.startswith("s_barrier") for l in lines[first:end]), name
            at, tiles[name] = end, tiles[name] + 1
        assert sum(l.startswith("s_barrier") for l in lines) == tiles[name], name
    assert sorted(tiles.values()) == [1] * 7 + [3], tiles
    for m in re.finditer(r"\.amdhsa_kernel (_ZN3moe\d+gg_f32_(?:split_|split_bwd_)?kernel\w+)(.*?)\.end_amdhsa_kernel", ffn_asm, re.S):
        assert re.search(r"\.amdhsa_private_segment_fixed_size 0\b", m.group(2)), m.group(1)
