#!/usr/bin/env python3
"""Generates mosaic_w4_tile.inc (greedy) and mosaic_w4_tile_sample.inc (sampling): one vocabulary tile of the 4-wave
fused kernel as one inline-asm statement, the hand-scheduled K-loop followed by the tile's vocabulary reduction, for
each width of the row tile (32*NB tokens, NB = 1..8, chosen by `if constexpr`).

The K-loop covers the nk K-tiles of the vocabulary tile.  Per K-tile (step g) a wave issues 16*nb
v_mfma_f32_16x16x32_bf16: its 128 vocabulary ids (8 blocks) against its half of the tokens (nb blocks), both K-halves of
the tile.  Up to nb = 4 (build) one K-half after the other, in two groups of 8*nb; between the MFMAs of a group sit the
ds_read_b128 that fetch the next group's fragments and the group's direct-to-LDS copies, so that nothing but MFMAs is
ever waited on in steady state.  The steady-state body (1 <= g, g + DEPTH < total) contains no branch at all -- a taken
branch costs more than one 16-cycle MFMA -- and all slot / pointer book-keeping is s_cselect arithmetic; the first step
and the last DEPTH run a guarded copy of the same schedule.  From nb = PAIRS_FROM on (build_pairs) both halves of a block
back to back; there every step is a steady one.

A ring holds DEPTH + 1 LM-head slots of 32 KiB and DEPTH hidden slots of 4*nb KiB.  DEPTH is two from nb = 3 on (nb = 8
fills the 160 KiB); one or two token blocks leave room for a third K-tile under way, which the copies need there,
because such a launch runs at the speed of memory.
"""
import os
import re
import sys

# Fragments by number: v[112:239].  The reduction's 32 logits and its temporaries alias the first of them, so that the
# compiler keeps 128 registers for what lives across a tile (with both as operands it spills).
FRAG_BASE = 112
# Up to four token blocks: a double buffer of 16 tuples, the LM head's eight first
FA = [[f"v[{FRAG_BASE + (b * 16 + i) * 4}:{FRAG_BASE + (b * 16 + i) * 4 + 3}]" for i in range(8)] for b in range(2)]
FB = [[f"v[{FRAG_BASE + (b * 16 + 8 + j) * 4}:{FRAG_BASE + (b * 16 + 8 + j) * 4 + 3}]" for j in range(8)] for b in range(2)]
VT0, VT1 = "%[vt0]", "%[vt1]"
VW, VH = ("%[vt0]", "%[vt2]"), ("%[vt1]", "%[vt3]")     # pair order: addresses of an LM-head and a hidden row, per K-half
WSRC, HSRC = "s[96:97]", "s[98:99]"
KT = "s95"
NK128 = "s94"

lines = []
uid = [0]
PAIRS_FROM = 5            # token blocks from which on the K-loop is in pair order (build_pairs)
SHAPE = {"nb": 8,         # token blocks of 16 per wave
         "tight": True}   # sampling: a quad that passes the column's bound is held against its own (off: for comparison)


def nb():
    return SHAPE["nb"]


def pairs():
    return nb() >= PAIRS_FROM


def depth():
    return 3 if nb() <= 2 else 2


def w_ring():
    return (depth() + 1) * 0x8000


def h_slot():
    return nb() * 0x1000


def h_ring():
    return depth() * h_slot()


def e(s):
    lines.append(s)


def label(name):
    uid[0] += 1
    return f"L{name}{uid[0]}_%="


# Accumulators, the AGPR file by number: block (bi, bj) = a[(bi*nb + bj)*4 .. +3].
def acc_block(bi, bj):
    base = (bi * nb() + bj) * 4
    return f"a[{base}:{base + 3}]"


def acc_reg(bi, bj, r):
    return f"a{(bi * nb() + bj) * 4 + r}"


def mfma(bi, bj, buf):
    e(f"v_mfma_f32_16x16x32_bf16 {acc_block(bi, bj)}, {FA[buf][bi]}, {FB[buf][bj]}, {acc_block(bi, bj)}")


def read_addr(ks):
    e(f"v_add_u32 {VT0}, %[wrd], %[rdw{ks}]")
    e(f"v_add_u32 {VT1}, %[hrd], %[rdh{ks}]")


def reads(buf):
    out = []
    for i in range(8):
        off = f" offset:{2048 * i}" if i else ""
        out.append(f"ds_read_b128 {FA[buf][i]}, {VT0}{off}")
    for j in range(nb()):
        off = f" offset:{2048 * j}" if j else ""
        out.append(f"ds_read_b128 {FB[buf][j]}, {VT1}{off}")
    return out


def dma_w(i):
    # the place of piece i within the wave's 8 KiB, exclusive-or the order of this unit's copies, which %[wdst] brings along
    return [f"s_xor_b32 m0, %[wdst], {1024 * i}", "s_nop 0", f"global_load_lds_dwordx4 %[woff{i}], {WSRC}"]


def dma_h(i):
    return [f"s_add_u32 m0, %[hdst], {w_ring() + 1024 * i}", "s_nop 0", f"global_load_lds_dwordx4 %[hoff{i}], {HSRC}"]


def dma_split(i, hidden):
    """the same copy as (m0 setup, the load): in the steady state the setup sits one MFMA ahead of the load, which
    supplies the wait state an M0 write needs before a direct-to-LDS load"""
    seq = dma_h(i) if hidden else dma_w(i)
    return seq[0], seq[2]


def next_slot(dst, slot, ring):
    """`dst` (a slot's offset plus this wave's share of it) to the ring's next slot"""
    if ring == 2 * slot and slot & (slot - 1) == 0:
        return [f"s_xor_b32 %[{dst}], %[{dst}], {hex(slot)}"]
    return [f"s_add_u32 %[{dst}], %[{dst}], {hex(slot)}",
            f"s_cmp_ge_u32 %[{dst}], {hex(ring)}",
            f"s_cselect_b32 vcc_lo, {hex(ring)}, 0",
            f"s_sub_u32 %[{dst}], %[{dst}], vcc_lo"]


def advance_h_ops():
    """next hidden copy: k index, source pointer (forward 128 bytes, back nk*128 after the last K-tile), slot"""
    return ["s_add_u32 %[hk], %[hk], 1",
            "s_add_u32 s98, s98, 128",
            "s_addc_u32 s99, s99, 0",
            "s_cmp_eq_u32 %[hk], %[nk]",
            f"s_cselect_b32 vcc_lo, {NK128}, 0",
            "s_cselect_b32 %[hk], 0, %[hk]",
            "s_sub_u32 s98, s98, vcc_lo",
            "s_subb_u32 s99, s99, 0"] + next_slot("hdst", h_slot(), h_ring())


def advance_w_ops():
    """next LM-head copy: k index, source pointer (forward 128 bytes or on to the next 256 rows), slot"""
    return ["s_add_u32 %[wk], %[wk], 1",
            "s_cmp_eq_u32 %[wk], %[nk]",
            "s_cselect_b32 vcc_lo, %[wwrap], 128",
            "s_cselect_b32 %[wk], 0, %[wk]",
            "s_add_u32 s96, s96, vcc_lo",
            "s_addc_u32 s97, s97, 0"] + next_slot("wdst", 0x8000, w_ring())


def rotate_read_slots_ops():
    ops = ["s_add_u32 %[wrd], %[wrd], 0x8000",
           f"s_cmp_ge_u32 %[wrd], {hex(w_ring())}",
           "s_cselect_b32 %[wrd], 0, %[wrd]"]
    if depth() == 2 and h_slot() & (h_slot() - 1) == 0:
        return ops + [f"s_xor_b32 %[hrd], %[hrd], {hex(h_slot())}"]
    return ops + [f"s_add_u32 %[hrd], %[hrd], {hex(h_slot())}",
                  f"s_cmp_ge_u32 %[hrd], {hex(h_ring())}",
                  "s_cselect_b32 %[hrd], 0, %[hrd]"]


def read_addr_ops(ks):
    return [f"v_add_u32 {VT0}, %[wrd], %[rdw{ks}]", f"v_add_u32 {VT1}, %[hrd], %[rdh{ks}]"]


def advance_h():
    for x in advance_h_ops():
        e(x)


def advance_w():
    for x in advance_w_ops():
        e(x)


def rotate_read_slots():
    for x in rotate_read_slots_ops():
        e(x)


def cond_g_ge1_and(plus):
    """scc = (g >= 1) && (g + plus < total)"""
    e(f"s_add_u32 vcc_lo, %[g], {plus}")
    e("s_cmp_lt_u32 vcc_lo, %[total]")
    e("s_cselect_b32 vcc_lo, 1, 0")
    e("s_cmp_ge_u32 %[g], 1")
    e("s_cselect_b32 vcc_hi, 1, 0")
    e("s_and_b32 vcc_lo, vcc_lo, vcc_hi")


def cond_plus(plus):
    """scc = (g + plus < total)"""
    e(f"s_add_u32 vcc_lo, %[g], {plus}")
    e("s_cmp_lt_u32 vcc_lo, %[total]")


def copy_pos(copies):
    """positions of a group's copies: spread over the group's first half or, where that is too short, over all of it"""
    n = 8 * nb()
    step = max(1, n // 2 // copies)
    return [min(1, n - copies) + i * step for i in range(copies)]


def read_pos(rd):
    """fragment reads by the MFMA they follow: one after each even MFMA, or as many a gap as a short group needs"""
    n = 8 * nb()
    at = {}
    for i, x in enumerate(rd or []):
        at.setdefault(min(2 * i, n - 2) if len(rd) * 2 <= n + 1 else i * n // len(rd), []).append(x)
    return at


def scheduled_group(buf, fill):
    """8*nb MFMAs on fragment buffer `buf`; fill[k] = the instructions that follow MFMA k.  A wave is alone on its
    SIMD and issues one instruction every few cycles, so whatever sits between two MFMAs beyond ~3 instructions
    delays the second one: the steady state keeps the gaps as short as the group's length allows."""
    order = [(bi, bj) for bi in range(8) for bj in range(nb())]
    for k in range(8 * nb()):
        mfma(*order[k], buf)
        for x in fill.get(k, []):
            e(x)


def group(buf, rd=None, dma=None, cond=None, after=None):
    """8*nb MFMAs on fragment buffer `buf` for the guarded (first / last steps) path.  rd = the ds_reads, spread over
    the group.  dma = copy sequences, copy i after MFMA pos[i]; guarded by `cond` when given (then the guarded
    span is pos[0]..pos[-1]); `after` runs once the copies are out."""
    e("s_waitcnt lgkmcnt(0)")
    n = 8 * nb()
    order = [(bi, bj) for bi in range(8) for bj in range(nb())]
    at = read_pos(rd)

    def step(k):
        mfma(*order[k], buf)
        for x in at.get(k, []):
            e(x)
    if not dma:
        for k in range(n):
            step(k)
        return
    pos = copy_pos(len(dma))
    lo, hi = pos[0], pos[-1]
    for k in range(lo):
        step(k)

    def span(with_dma):
        for k in range(lo, hi + 1):
            step(k)
            if with_dma and k in pos:
                for x in dma[pos.index(k)]:
                    e(x)
        if with_dma and after:
            after()
    if cond is None:
        span(True)
    else:
        skip, join = label("nodma"), label("join")
        cond()
        e(f"s_cbranch_scc0 {skip}")
        span(True)
        e(f"s_branch {join}")
        e(f"{skip}:")
        span(False)
        e(f"{join}:")
    for k in range(hi + 1, n):
        step(k)


def steady_fill(buf):
    """Gap contents of one steady-state group: the fragment reads of the other buffer, the copies, and the scalar
    book-keeping behind them."""
    copies = nb() if buf == 1 else 8
    split = [dma_split(i, hidden=(buf == 1)) for i in range(copies)]
    rd = reads(1 - buf)
    if buf == 0:
        # the read slots of the NEXT tile, ahead of the sync, and the addresses of its first-half fragments
        ops = [advance_w_ops(), rotate_read_slots_ops(), read_addr_ops(0)]
    else:
        # next step's second-half fragment addresses;
        # scc = (k-tile index < nk) && (g + depth < total): the next step belongs to this statement and is steady
        ops = [advance_h_ops(), ["s_add_u32 %[g], %[g], 1", f"s_add_u32 {KT}, {KT}, 1"], read_addr_ops(1)]
    last = ["s_add_u32 vcc_lo, %[g], " + str(depth()), "s_cmp_lt_u32 vcc_lo, %[total]",
            "s_cselect_b32 vcc_lo, %[nk], 0", f"s_cmp_lt_u32 {KT}, vcc_lo"] if buf == 1 else []
    fill = {}
    # evenly over the gaps; a read sits between a copy's M0 write and its load
    seq = []
    for i, x in enumerate(rd):
        seq += [split[i][0], x, split[i][1]] if i < copies else [x]
    seq += [x for part in ops for x in part] + last
    n = 8 * nb()
    for i, x in enumerate(seq):
        fill.setdefault(i * n // len(seq), []).append(x)
    return fill


def step_end(top):
    e("s_add_u32 %[g], %[g], 1")
    e(f"s_add_u32 {KT}, {KT}, 1")
    e(f"s_cmp_lt_u32 {KT}, %[nk]")
    e(f"s_cbranch_scc1 {top}")


LOG2E = 0x3FB8AA3B        # fp32 1.4426950408889634
NEG_LOG2E = 0xBFB8AA3B
X = [f"v{FRAG_BASE + i}" for i in range(32)]
ET, _, ENML, EY, ESEL = (f"v{FRAG_BASE + 32 + k}" for k in range(5))
MASK = ["s[88:89]", "s[90:91]", "s[92:93]"]


def own_maximum(M):
    """M = ET, the column's largest logit, -2^100 at least, and ENML = -M log2 e: a lane whose 32 ids are all at minus
    infinity is then an empty one (x - M never is inf - inf), as it is to the merges, and a NaN shows in the sum alone."""
    e(f"v_max_f32 {M}, {hex(KNEG)}, {ET}")
    e(f"v_mul_f32 {ENML}, {hex(NEG_LOG2E)}, {M}")


def tile_exponentials(XS, S):
    """S = sum of 2^(x log2 e + ENML) over the column's 32 logits, in four chains"""
    for el in range(32):
        e(f"v_fmamk_f32 {XS[el]}, {XS[el]}, {hex(LOG2E)}, {ENML}")
    for el in range(32):
        e(f"v_exp_f32 {XS[el]}, {XS[el]}")
    for step in range(1, 8):
        for r in range(4):
            e(f"v_add_f32 {XS[r]}, {XS[r]}, {XS[4 * step + r]}")
    e(f"v_add_f32 {XS[0]}, {XS[0]}, {XS[1]}")
    e(f"v_add_f32 {XS[2]}, {XS[2]}, {XS[3]}")
    e(f"v_add_f32 {S}, {XS[0]}, {XS[2]}")


def reduce_column(tb):
    """The vocabulary reduction of one token column of the finished tile (this lane: 8 blocks x 4 ids, element
    e = 4*bi + r is vocabulary id vb + 16*bi + r) to its own (max, sum-exp, arg-max), which the kernel folds into the
    running ones:
        t = max_e x[e];  sel = lowest e with x[e] == t;  i = vb + code(sel)
        m = max(t, -2^100);  s = sum_e 2^(x[e] log2 e - m log2 e)
    Written so that no instruction needs a wait state: a comparison result is consumed three instructions later
    (three SGPR pairs in rotation), an exponential at the earliest two instructions later."""
    M, S, I = f"%[m{tb}]", f"%[s{tb}]", f"%[i{tb}]"
    for el in range(32):
        e(f"v_accvgpr_read_b32 {X[el]}, {acc_reg(el // 4, tb, el % 4)}")
    e(f"v_max3_f32 {ET}, {X[0]}, {X[1]}, {X[2]}")
    for j in range(14):
        e(f"v_max3_f32 {ET}, {ET}, {X[3 + 2 * j]}, {X[4 + 2 * j]}")
    e(f"v_max_f32 {ET}, {ET}, {X[31]}")
    # lowest element attaining the maximum: descending scan, a lower match overwrites a higher one
    e(f"v_mov_b32 {ESEL}, 0")
    order = list(range(31, -1, -1))
    pending = []
    for n, el in enumerate(order):
        mask = MASK[n % 3]
        e(f"v_cmp_eq_f32_e64 {mask}, {X[el]}, {ET}")
        pending.append((mask, el))
        if len(pending) == 3:
            mk, pe = pending.pop(0)
            e(f"v_cndmask_b32_e64 {ESEL}, {ESEL}, {pe}, {mk}")
    own_maximum(M)                                    # and two selects are still pending
    for mk, pe in pending:
        e(f"v_cndmask_b32_e64 {ESEL}, {ESEL}, {pe}, {mk}")
    e(f"v_lshrrev_b32 {EY}, 2, {ESEL}")               # code = 16 * (sel / 4) + sel % 4
    e(f"v_and_b32 {ESEL}, 3, {ESEL}")
    e(f"v_lshl_add_u32 {ESEL}, {EY}, 4, {ESEL}")
    e(f"v_add_u32 {I}, %[vb], {ESEL}")
    tile_exponentials(X, S)


# ---- the sampling statement (Gumbel-max at temperature tau; noise from Philox4x32-10 keyed by seed, counter =
# (vocabulary id / 4, position, 0, 0), word id % 4).  Its registers beyond the
# greedy reduction's are fragment registers that are dead by then: v[164:171] two generations of the generator's two
# 64-bit products, v[172:173] the per-column product, v[174:179] temporaries of the rare exact path, v[184:215] the ids' part.
PHILOX_M0, PHILOX_M1 = "%[pm0]", "%[pm1]"
KNEG = 0xF1800000          # -2^100
TWO23_101 = 0x4B0147AE     # 2^23 * 1.01
TWO23 = 0x4B000000
NEG_LN2 = 0xBF317218
TWO_M23 = 0x34000000
TWO_M8 = 0x3B800000
THIRD = 0x3EAAAAAB
slow_blocks = []
# The reduction's temporaries live in fragment registers that are dead by then, the generator's round keys in scalar
# registers the statement fills itself from the seed: neither costs the register allocator anything.
SAMPLE_TEMPS = {name: f"v{FRAG_BASE + 32 + k}" for k, name in enumerate(
    ("et", "unused", "enml", "ey", "yt", "xsel", "sels", "wlo", "wm", "v4b", "v4q", "a0", "sw16", "sw32", "sw48", "pw", "px", "pe", "cnt", "nq"))}
SAMPLE_TEMPS.update(best="v180", wq="v181")
KEY0_BASE, KEY1_BASE = 68, 78
SAMPLE_TEMPS.update({f"k0_{r}": f"s{KEY0_BASE + r}" for r in range(10)})
SAMPLE_TEMPS.update({f"k1_{r}": f"s{KEY1_BASE + r}" for r in range(10)})


# What of the first rounds depends on the ids alone is the same for every column of the tile, four registers per quad: the
# counter is (v4, position, 0, 0), so round 0 multiplies v4 alone (the second product is zero), of round 1's products one has
# the position alone and one v4 alone, and of round 2's the first v4 alone.  Kept: round 0's low half; round 1's low half xored
# with round 2's key; round 2's high half xored with its key, and its low half.
ID_BASE = 184


def id_reg(bi, k):
    return f"v{ID_BASE + 4 * bi + k}"


def philox_ids():
    """The ids' part of the generator, once a tile: three of a quad's eighteen products and four of its other instructions.
    A wave is alone on its SIMD and issues an instruction every 4.6 cycles, the 64-bit product like any other, so what
    counts is how many there are: 42 a quad with this in every column, 36 without."""
    for bi in range(8):
        low, b1, hi2, lo2 = (id_reg(bi, k) for k in range(4))
        e(f"v_add_u32 %[v4q], {4 * bi}, %[v4b]")
        e(f"v_mad_u64_u32 v[164:165], vcc, {PHILOX_M0}, %[v4q], 0")      # round 0: lo -> a3, hi
        e(f"v_xor_b32 v165, %[k1_0], v165")                              # a2 = hi ^ k1
        e(f"v_mov_b32 {low}, v164")
        e(f"v_mad_u64_u32 v[166:167], vcc, {PHILOX_M1}, v165, 0")        # round 1, second product: lo -> b1, hi
        e(f"v_xor_b32 v167, %[k0_1], v167")                              # b0 = hi ^ k0   (a1 = 0)
        e(f"v_xor_b32 {b1}, %[k0_2], v166")
        e(f"v_mad_u64_u32 v[168:169], vcc, {PHILOX_M0}, v167, 0")        # round 2, first product
        e(f"v_xor_b32 {hi2}, %[k1_2], v169")
        e(f"v_mov_b32 {lo2}, v168")


def philox_quad(tb, bi, XS):
    """Words of the four ids vb + 16*bi .. +3 of column tb's position, and the jump to the exact path when one of
    them could still win.  Begins in round 1, with the ids' part (philox_ids) and the product of the position alone (per
    column, in v[172:173], its high half already xored with the round key)."""
    A, B, C, D = ("v164", "v165"), ("v166", "v167"), ("v168", "v169"), ("v170", "v171")
    pair = lambda r: f"v[{r[0][1:]}:{r[1][1:]}]"
    low, b1, hi2, lo2 = (id_reg(bi, k) for k in range(4))
    e(f"v_xor_b32 {A[1]}, v173, {low}")                              # b2 = (hi(M0 a0) ^ k1) ^ a3
    e(f"v_mad_u64_u32 {pair(B)}, vcc, {PHILOX_M1}, {A[1]}, 0")       # round 2, second product
    e(f"v_xor_b32 {B[1]}, {b1}, {B[1]}")                             # hi ^ b1 ^ k0
    e(f"v_xor_b32 {A[1]}, v172, {hi2}")                              # hi(M0 b0) ^ b3 ^ k1, b3 = lo(M0 a0)
    c0, c1, c2, c3 = B[1], B[0], A[1], lo2
    cur, nxt = (A, B), (C, D)
    for r in range(3, 10):
        PA, PB = nxt
        e(f"v_mad_u64_u32 {pair(PA)}, vcc, {PHILOX_M0}, {c0}, 0")
        e(f"v_mad_u64_u32 {pair(PB)}, vcc, {PHILOX_M1}, {c2}, 0")
        e(f"v_bitop3_b32 {PB[1]}, {PB[1]}, {c1}, %[k0_{r}] bitop3:0x96")     # truth table 0x96: a ^ b ^ c
        e(f"v_bitop3_b32 {PA[1]}, {PA[1]}, {c3}, %[k1_{r}] bitop3:0x96")
        c0, c1, c2, c3 = PB[1], PB[0], PA[1], PA[0]
        cur, nxt = nxt, cur
    words = [c0, c1, c2, c3]
    # a word below the column's bound cannot win: only 2^-23-sized tails of the uniform reach the running best
    e(f"v_max3_u32 %[wm], {words[0]}, {words[1]}, {words[2]}")
    e(f"v_max_u32 %[wm], %[wm], {words[3]}")
    e(f"v_cmp_ge_u32 vcc, %[wm], %[wlo]")
    slow, flush, back = label(f"slow{tb}{bi}"), label(f"flush{tb}{bi}"), label(f"back{tb}{bi}")
    e(f"s_cbranch_vccnz {slow}")
    e(f"{back}:")
    # Out of line: some lane holds a candidate.  Its word, logit and element go into the lane's one-deep queue, to be
    # scored once at the end of the column.  When a lane would queue a second one, the queues are scored and emptied
    # first; when that lane's two candidates are both of this quad, the quad's four ids are scored directly.
    M3, M2, M1, SINK = MASK[0], MASK[1], MASK[2], "s[66:67]"
    els = [bi * 4 + r for r in range(4)]
    queue, full = label(f"queue{tb}{bi}"), label(f"full{tb}{bi}")
    passes = [f"v_cmp_ge_u32_e64 {M3}, {words[3]}, %[wlo]",
              f"v_cmp_ge_u32_e64 {M2}, {words[2]}, %[wlo]",
              f"v_cmp_ge_u32_e64 {M1}, {words[1]}, %[wlo]"]
    if SHAPE["tight"]:
        # The quad's own bound: its four logits against the best score known by now.  The column's bound, made of the
        # lane's largest logit of 32 and the best score before the tile, passes nearly every quad of a unit's first
        # tiles in some lane; this one leaves a few, and 11 instructions take the place of 35 to 200.
        xs = [XS[x] for x in els]
        own = [f"v_max3_f32 v174, {xs[0]}, {xs[1]}, {xs[2]}", f"v_max_f32 v174, v174, {xs[3]}"]
        own += word_bound("v174", "%[best]", "v175", "%[wq]")
        own += [f"v_cmp_ge_u32 vcc, %[wm], %[wq]", f"s_cbranch_vccz {back}"]
        passes = [ln.replace("%[wlo]", "%[wq]") for ln in passes]
    else:
        own = []
    low = "%[wq]" if SHAPE["tight"] else "%[wlo]"
    blk = [f"{slow}:"] + own + passes + [
           f"v_cmp_ge_u32 vcc, {words[0]}, {low}",
           f"v_addc_co_u32_e64 %[nq], {SINK}, 0, 0, {M3}",               # candidates of this quad, per lane
           f"v_addc_co_u32_e64 %[nq], {SINK}, 0, %[nq], {M2}",
           f"v_addc_co_u32_e64 %[nq], {SINK}, 0, %[nq], {M1}",
           f"v_addc_co_u32_e64 %[nq], {SINK}, 0, %[nq], vcc",
           f"v_add_u32 %[cnt], %[cnt], %[nq]",
           f"v_cmp_lt_u32 vcc, 1, %[cnt]",
           f"s_cbranch_vccnz {flush}",
           f"{queue}:",
           f"v_cmp_ge_u32 vcc, {words[0]}, {low}"]
    for mk, r in ((M3, 3), (M2, 2), (M1, 1)):
        blk += [f"v_cndmask_b32_e64 %[pw], %[pw], {words[r]}, {mk}",
                f"v_cndmask_b32_e64 %[px], %[px], {XS[els[r]]}, {mk}",
                f"v_cndmask_b32_e64 %[pe], %[pe], {els[r]}, {mk}"]
    blk += [f"v_cndmask_b32 %[pw], %[pw], {words[0]}, vcc",
            f"v_cndmask_b32 %[px], %[px], {XS[els[0]]}, vcc",
            f"v_cndmask_b32_e64 %[pe], %[pe], {els[0]}, vcc",
            f"s_branch {back}",
            f"{flush}:"]
    if SHAPE["tight"]:                     # nothing to score where no lane's queue held anything
        nothing = label(f"nothing{tb}{bi}")
        blk += ["v_cmp_ne_u32 vcc, %[cnt], %[nq]", f"s_cbranch_vccz {nothing}"]
        blk += score_candidate("%[pw]", "%[px]", "%[pe]") + empty_queue() + share_best() + [f"{nothing}:"]
    else:
        blk += score_candidate("%[pw]", "%[px]", "%[pe]") + empty_queue()
    blk += [f"v_cmp_lt_u32 vcc, 1, %[nq]",
            f"s_cbranch_vccnz {full}"]
    blk += passes + ["v_mov_b32 %[cnt], %[nq]", f"s_branch {queue}", f"{full}:"]
    for r in range(3, -1, -1):
        blk += score_candidate(words[r], XS[els[r]], str(els[r]))
    blk += (["v_mov_b32 %[cnt], 0"] + share_best() if SHAPE["tight"] else []) + [f"s_branch {back}"]
    slow_blocks.append(blk)


def word_bound(x, best, tmp, out):
    """the lowest word of a logit up to x that can still win against the score `best`: candidates have
    (w >> 9) >= 2^23 - Z, Z = min(2^23, 1.01 * 2^23 * exp((x - best) / tau) + 2)"""
    return [f"v_sub_f32 {tmp}, {x}, {best}",
            f"v_mul_f32 {tmp}, %[itl], {tmp}",                           # log2(e) / tau
            f"v_exp_f32 {tmp}, {tmp}",
            "s_nop 0",
            f"v_mul_f32 {tmp}, {hex(TWO23_101)}, {tmp}",
            f"v_add_f32 {tmp}, 2.0, {tmp}",
            f"v_min_f32 {tmp}, {hex(TWO23)}, {tmp}",
            f"v_cvt_u32_f32 {out}, {tmp}",
            f"v_sub_u32 {out}, {hex(0x800000)}, {out}",
            f"v_lshlrev_b32 {out}, 9, {out}"]


def share_best():
    """the best score known of the token: what its four lanes have scored in this tile, and the best before it"""
    return ["ds_bpermute_b32 v177, %[sw16], %[yt]",
            "ds_bpermute_b32 v178, %[sw32], %[yt]",
            "ds_bpermute_b32 v179, %[sw48], %[yt]",
            "v_max_f32 %[best], %[best], %[yt]",
            "s_waitcnt lgkmcnt(0)",
            "v_max3_f32 %[best], %[best], v177, v178",
            "v_max_f32 %[best], %[best], v179"]


def empty_queue():
    return ["v_mov_b32 %[cnt], 0", "v_mov_b32 %[pw], 0", f"v_mov_b32 %[px], {hex(KNEG)}", "v_mov_b32 %[pe], 0"]


def score_candidate(word, x, el):
    """y = x + tau * g(u) of one id per lane (u from the id's word, g = -ln(-ln u), next to u = 1 by the series of
    -ln(1 - e)), and the tile's best (score, element, logit) updated by it: a higher score wins, the lower element
    on equal scores."""
    M3, M2, M1 = MASK
    return [f"v_lshrrev_b32 v174, 9, {word}",                            # k
            f"v_sub_u32 v175, {hex(0x7FFFFF)}, v174",                    # 2^23 - 1 - k
            "v_cvt_f32_u32 v174, v174",
            "v_cvt_f32_u32 v175, v175",
            "v_add_f32 v174, 0.5, v174",
            "v_add_f32 v175, 0.5, v175",
            f"v_mul_f32 v174, {hex(TWO_M23)}, v174",                     # u
            f"v_mul_f32 v175, {hex(TWO_M23)}, v175",                     # e = 1 - u
            "v_log_f32 v176, v174",
            f"v_mul_f32 v177, {hex(THIRD)}, v175",                       # e (1 + e (1/2 + e/3)) = -ln(1 - e) near u = 1
            "v_add_f32 v177, 0.5, v177",
            f"v_mul_f32 v176, {hex(NEG_LN2)}, v176",                     # -ln u
            "v_mul_f32 v177, v175, v177",
            "v_add_f32 v177, 1.0, v177",
            f"v_cmp_gt_f32 vcc, {hex(TWO_M8)}, v175",
            "v_mul_f32 v177, v175, v177",
            "s_nop 0",
            "v_cndmask_b32 v176, v176, v177, vcc",                       # inner = e < 2^-8 ? series : by the logarithm
            "v_log_f32 v176, v176",
            "s_nop 0",
            f"v_mul_f32 v176, {hex(NEG_LN2)}, v176",                     # g = -ln(inner)
            "v_mul_f32 v176, %[tau], v176",
            f"v_add_f32 v176, {x}, v176",                                # y = x + tau g
            f"v_cmp_eq_f32_e64 {M2}, v176, %[yt]",
            f"v_cmp_gt_u32_e64 {M1}, %[sels], {el}",
            "v_cmp_gt_f32 vcc, v176, %[yt]",
            "s_nop 1",
            f"s_and_b64 {M2}, {M2}, {M1}",
            f"s_or_b64 vcc, vcc, {M2}",
            "s_nop 1",
            f"v_cndmask_b32_e64 %[sels], %[sels], {el}, vcc",
            f"v_cndmask_b32 %[xsel], %[xsel], {x}, vcc",
            "v_cndmask_b32 %[yt], %[yt], v176, vcc"]


def reduce_column_sample(tb):
    """Column tb of the finished tile under sampling: (max, sum-exp) as in the greedy reduction, and the running
    arg-max of x + tau*g with the plain logit there.  Exact: an id is skipped only when its uniform lies below what
    the best score seen so far minus the column's largest logit of this tile demands (1 - u < exp((t - ym) / tau),
    taken with a 1% margin), which no winner can."""
    M, S, I, YM, XA, POS = (f"%[m{tb}]", f"%[s{tb}]", f"%[i{tb}]", f"%[ym{tb}]", f"%[xa{tb}]", f"%[pos{tb}]")
    XS = [f"v{FRAG_BASE + i}" for i in range(32)]
    # the best score so far of the three other lanes that hold the same token (lane ^ 16, ^ 32, ^ 48): any score
    # already reached for the row bounds what can still win it
    e(f"ds_bpermute_b32 v177, %[sw16], {YM}")
    e(f"ds_bpermute_b32 v178, %[sw32], {YM}")
    e(f"ds_bpermute_b32 v179, %[sw48], {YM}")
    for el in range(32):
        e(f"v_accvgpr_read_b32 {XS[el]}, {acc_reg(el // 4, tb, el % 4)}")
    e(f"v_max3_f32 {ET}, {XS[0]}, {XS[1]}, {XS[2]}")
    for j in range(14):
        e(f"v_max3_f32 {ET}, {ET}, {XS[3 + 2 * j]}, {XS[4 + 2 * j]}")
    e(f"v_max_f32 {ET}, {ET}, {XS[31]}")
    # the bound on the words: candidates have (w >> 9) >= 2^23 - Z, Z = min(2^23, 1.01 * 2^23 * exp((t - ym)/tau) + 2)
    e("s_waitcnt lgkmcnt(0)")
    e(f"v_max3_f32 v177, v177, v178, v179")
    e(f"v_max_f32 v177, v177, {YM}")
    if SHAPE["tight"]:
        e("v_mov_b32 %[best], v177")
    e(f"v_sub_f32 {EY}, {ET}, v177")
    e(f"v_mul_f32 {EY}, %[itl], {EY}")                               # log2(e) / tau
    e(f"v_exp_f32 {EY}, {EY}")
    e(f"v_xor_b32 %[a0], %[k0_0], {POS}")                            # round 0: a0 = position ^ k0
    e(f"v_mul_f32 {EY}, {hex(TWO23_101)}, {EY}")
    e(f"v_mad_u64_u32 v[172:173], vcc, {PHILOX_M0}, %[a0], 0")       # round 1, first product: position only
    e(f"v_add_f32 {EY}, 2.0, {EY}")
    e(f"v_min_f32 {EY}, {hex(TWO23)}, {EY}")
    e(f"v_cvt_u32_f32 %[wlo], {EY}")
    e(f"v_xor_b32 v173, %[k1_1], v173")
    e(f"v_sub_u32 %[wlo], {hex(0x800000)}, %[wlo]")
    e(f"v_lshlrev_b32 %[wlo], 9, %[wlo]")
    e(f"v_mov_b32 %[yt], {hex(KNEG)}")
    e("v_mov_b32 %[sels], 0")
    e(f"v_mov_b32 %[xsel], 0")
    for ln in empty_queue():
        e(ln)
    # a quad is 264 bytes, in which the rounds' 8-byte instructions follow 20: they are to lie on 8-byte boundaries (where they
    # do not, 16000 rows of 32000 x 1024 take 976 us instead of 953, 4096 rows of 126464 x 4096 2878 instead of 2851)
    e(".p2align 3")
    e("s_nop 0")
    for bi in range(7, -1, -1):
        philox_quad(tb, bi, XS)
    empty = label(f"empty{tb}")
    e("v_cmp_ne_u32 vcc, 0, %[cnt]")                                 # what is left in the queues, if anything
    e(f"s_cbranch_vccz {empty}")
    for ln in score_candidate("%[pw]", "%[px]", "%[pe]"):
        e(ln)
    e(f"{empty}:")
    # the tile's best against the running best (strict: an equal score in a later tile has a higher id)
    e(f"v_cmp_gt_f32 vcc, %[yt], {YM}")
    e(f"v_lshrrev_b32 {EY}, 2, %[sels]")
    e(f"v_and_b32 %[sels], 3, %[sels]")
    e(f"v_lshl_add_u32 %[sels], {EY}, 4, %[sels]")
    e(f"v_add_u32 %[sels], %[vb], %[sels]")
    e(f"v_cndmask_b32 {I}, {I}, %[sels], vcc")
    e(f"v_cndmask_b32 {XA}, {XA}, %[xsel], vcc")
    e(f"v_cndmask_b32 {YM}, {YM}, %[yt], vcc")
    own_maximum(M)
    tile_exponentials(XS, S)


# %[first] = TAKE asks for it.
TAKE = 0x80000000


def take_published():
    """The best scores that other units have published for this wave's rows (the kernel says how, at its shared bounds) into
    the columns' running best, as a float just below.  Here, between the tile's products and its draw, a unit's second tile
    finds what the first ones of all units have reached; ahead of the products, where it stood, they were still at it.
    %[rb]: the first of the rows' words, %[rl]: the last row that is there."""
    T = [f"v{FRAG_BASE + i}" for i in range(nb())]
    best = ["v180", "v181"][:(nb() + 3) // 4]
    e("v_mbcnt_lo_u32_b32 v176, -1, 0")
    e("v_mbcnt_hi_u32_b32 v176, -1, v176")
    for k, b in enumerate(best):                                     # lane group q: columns q and q + 4
        e(f"v_add_u32 {b}, {64 * k}, v176")
        e(f"v_min_i32 {b}, %[rl], {b}")
        e(f"v_lshlrev_b32 {b}, 2, {b}")
        e(f"global_load_dword {b}, {b}, %[rb] sc0")
    e("v_and_b32 v176, 15, v176")
    e("v_lshlrev_b32 v176, 2, v176")
    e("s_waitcnt vmcnt(0)")
    for b in best:                                                   # below, and back from the words' order (its own inverse)
        e(f"v_add_u32 {b}, -2, {b}")
        e(f"v_ashrrev_i32 v177, 31, {b}")
        e("v_lshrrev_b32 v177, 1, v177")
        e(f"v_xor_b32 {b}, v177, {b}")
    for tb in range(nb()):
        e(f"ds_bpermute_b32 {T[tb]}, v176, {best[tb // 4]} offset:{64 * (tb % 4)}")
    e("s_waitcnt lgkmcnt(0)")
    for tb in range(nb()):
        e(f"v_max_f32 %[ym{tb}], %[ym{tb}], {T[tb]}")


def build_tile_sample():
    """The statement of the sampling kernel: the K-loop, then the
    reduction with the noise; the rare exact paths sit behind the end of the statement."""
    slow_blocks.clear()
    build_loop(take_published)
    e(f"s_mov_b32 %[k0_0], %[seed_lo]")                              # key of round r = seed + r * (golden-ratio words)
    e(f"s_mov_b32 %[k1_0], %[seed_hi]")
    for r in range(1, 10):
        e(f"s_add_u32 %[k0_{r}], %[k0_{r - 1}], 0x9e3779b9")
        e(f"s_add_u32 %[k1_{r}], %[k1_{r - 1}], 0xbb67ae85")
    e("v_lshrrev_b32 %[v4b], 2, %[vb]")
    e("v_mbcnt_lo_u32_b32 %[sw16], -1, 0")                           # lane id, then the byte addresses of the lanes
    e("v_mbcnt_hi_u32_b32 %[sw16], -1, %[sw16]")                     # ^ 16, ^ 32, ^ 48 for the cross-lane reads
    e("v_xor_b32 %[sw32], 32, %[sw16]")
    e("v_xor_b32 %[sw48], 48, %[sw16]")
    e("v_xor_b32 %[sw16], 16, %[sw16]")
    e("v_lshlrev_b32 %[sw32], 2, %[sw32]")
    e("v_lshlrev_b32 %[sw48], 2, %[sw48]")
    e("v_lshlrev_b32 %[sw16], 2, %[sw16]")
    philox_ids()
    for tb in range(nb()):
        reduce_column_sample(tb)
    done = label("done")
    e(f"s_branch {done}")
    for blk in slow_blocks:
        for ln in blk:
            e(ln)
    e(f"{done}:")
    named = re.compile(r"%\[(\w+)\]")
    lines[:] = [named.sub(lambda m: SAMPLE_TEMPS.get(m.group(1), m.group(0)), ln) for ln in lines]


def build_tile():
    """The statement of the greedy kernel: the K-loop on accumulators it starts itself, then the reduction of the
    tile."""
    build_loop()
    for tb in range(nb()):
        reduce_column(tb)


def mask_counted(between=None):
    """The last tile of a vocabulary that is no multiple of 256 lies over the vocabulary's last 256 ids; those below
    %[first] belong to the tile before it and are taken out here: their logits become -2^100.  %[first] is 0 for every
    other tile.  One compare per element serves all columns; a compare's result is read two wait states later."""
    skip = label("whole")
    e("s_cmp_eq_u32 %[first], 0")
    e(f"s_cbranch_scc1 {skip}")
    if between:
        take = label("take")
        e(f"s_cmp_eq_u32 %[first], {hex(TAKE)}")
        e(f"s_cbranch_scc1 {take}")
    e(f"v_sub_u32 {ET}, %[first], %[vb]")             # elements with a code below it (signed) are taken out
    e(f"v_mov_b32 {EY}, {hex(KNEG)}")
    for el in range(32):
        e(f"v_cmp_lt_i32 vcc, {16 * (el // 4) + el % 4}, {ET}")
        for tb in range(nb()):
            e(f"v_accvgpr_read_b32 {X[tb]}, {acc_reg(el // 4, tb, el % 4)}")
        e("s_nop 1")
        for tb in range(nb()):
            e(f"v_cndmask_b32 {X[tb]}, {X[tb]}, {EY}, vcc")
        for tb in range(nb()):
            e(f"v_accvgpr_write_b32 {acc_reg(el // 4, tb, el % 4)}, {X[tb]}")
    if between:                                       # a whole tile too
        e(f"s_branch {skip}")
        e(f"{take}:")
        between()
    e(f"{skip}:")


def build_loop(between=None):
    """The width's K-loop, and what of its tile is not counted."""
    build_pairs() if pairs() else build()
    mask_counted(between)


def build():
    # entry: pointers into fixed SGPR pairs, first fragments of the current step
    e("s_mov_b32 s96, %[wsrc_lo]")
    e("s_mov_b32 s97, %[wsrc_hi]")
    e("s_mov_b32 s98, %[hsrc_lo]")
    e("s_mov_b32 s99, %[hsrc_hi]")
    e(f"s_add_u32 {NK128}, %[hwrap], 128")      # nk * 128
    e(f"s_mov_b32 {KT}, 0")
    read_addr(0)
    for r in reads(0):
        e(r)
    # the statement owns the accumulators: clear them while the first fragments are on their way (measured: writing a
    # tile's first products without an addend instead saves nothing)
    for i in range(32 * nb()):
        e(f"v_accvgpr_write_b32 a{i}, 0")
    e("s_nop 7")
    top, steady, generic, out = label("top"), label("steady"), label("generic"), label("out")
    e(f"{top}:")
    # Steady state (1 <= g and g + depth < total): every copy and the sync happen, no branch inside the body, one taken
    # branch per step (the back edge, issued right behind the last MFMA).
    cond_g_ge1_and(depth())
    e(f"s_cbranch_scc0 {generic}")
    read_addr(1)
    e(f"{steady}:")
    leave = label("leave")
    e("s_waitcnt lgkmcnt(0)")
    scheduled_group(0, steady_fill(0))                       # LM-head tile g + depth goes out
    # all copies of step g + 1 have landed: younger are the LM-head tiles of steps g + 2 .. g + depth and the hidden
    # tiles of steps g + 2 .. g + depth - 1; and this wave's fragments
    e(f"s_waitcnt vmcnt({8 * (depth() - 1) + nb() * (depth() - 2)}) lgkmcnt(0)")
    e("s_barrier")
    scheduled_group(1, steady_fill(1))                       # hidden tile g + depth goes out
    e(f"s_cbranch_scc1 {steady}")
    e(f"{leave}:")
    e(f"s_cmp_lt_u32 {KT}, %[nk]")
    e(f"s_cbranch_scc0 {out}")
    # First step and the last ones: same schedule with every part guarded.
    e(f"{generic}:")
    read_addr(1)
    group(0, rd=reads(1), dma=[dma_w(i) for i in range(8)], cond=lambda: cond_g_ge1_and(depth()), after=advance_w)
    nosync, stepend = label("nosync"), label("stepend")
    cond_plus(1)
    e(f"s_cbranch_scc0 {nosync}")
    e("s_waitcnt lgkmcnt(0)")
    e("s_waitcnt vmcnt(0)")       # outside the steady state no copy younger than step g+1 needs to stay in flight
    e("s_barrier")
    rotate_read_slots()
    read_addr(0)
    group(1, rd=reads(0), dma=[dma_h(i) for i in range(nb())], cond=lambda: cond_plus(depth()), after=advance_h)
    e(f"s_branch {stepend}")
    e(f"{nosync}:")
    group(1)
    e(f"{stepend}:")
    step_end(top)
    e(f"{out}:")
    # exit: no fragment read may still be in flight, results visible to the VALU, pointers back to the operands
    e("s_waitcnt lgkmcnt(0)")
    e("s_nop 15")
    e("s_nop 15")
    e("s_mov_b32 %[wsrc_lo], s96")
    e("s_mov_b32 %[wsrc_hi], s97")
    e("s_mov_b32 %[hsrc_lo], s98")
    e("s_mov_b32 %[hsrc_hi], s99")


# ---- The K-loop in pair order, for the widths whose time goes into the matrix cores.
#
# Under the power cap what a product costs is energy, and a product that accumulates where the one before it did costs
# less: its addend need not come out of the register file.  Register-only loops over 64 accumulator blocks: 2.02 PFLOP/s
# block after block with one K-half and then the other, 2.14 with the two halves of a block back to back (four or eight
# products of a block in a row: 2.12 to 2.15).  So a step (K-tile) here takes block after block, both halves of each:
# vocabulary block i = 0..7, under it the token blocks j = 0..nb-1, forward and backward in turn.  The sums run in the
# order of the other loop, so the results are the same bits.
#
# Fragments, in 32 tuples as there: the token blocks, which every row of blocks uses, lie in X_PAIRS pairs (both halves)
# and stay for a step, the vocabulary blocks pass through a ring of four pairs.  Up to six token blocks are double-
# buffered; of seven and eight the last (2 nb - 12) are read into the registers of the blocks that the last row of
# products, which runs backward, is done with.  The register numbers repeat every other step: two bodies.
#
# Rings, as deep as there: LM head three slots, hidden two.  The sync of a step (two rows in) publishes the next step's
# hidden tile, its vocabulary blocks 0..3 and this step's blocks 4..7; it frees this step's hidden tile (read whole by
# then), this step's blocks 0..3 and the last step's 4..7.  The waves that copy blocks 0..3 (the even ones) therefore run
# three K-tiles ahead and the odd ones two.  The copies are spread over the whole time from one sync to the next, the
# hidden tile's first, since only it has to land by the next sync.  Spread over two thirds of it 4096 rows took 0.4% more,
# 2077 rows 0.7%, one row tile at the speed of memory 3 to 7%; over less still 3 to 8%.
#
# Every step of a unit copies, also the last ones, into slots that nobody reads any more: of the LM head the last K-tile
# again, of the hidden rows what lies at the front of them.  A guarded form of the steps would be code that runs cold, a
# few steps a unit (measured: 0.3% slower).
#
# 4096 x 126464 x 4096: 2641 -> 2535 us, 2077 rows (width 6) 1484 -> 1411, 58524 rows 39.7 -> 37.3 ms (one box each, in
# turn with the other loop).
X_PAIRS = 12
Y_RING = 4


def x_slot(par, j):
    """where token block j of a step of this parity lies"""
    if 2 * nb() <= X_PAIRS:
        return par * nb() + j
    early = X_PAIRS - nb()
    if j < early:
        return par * early + j
    return 2 * early + (j - early if par == 0 else nb() - 1 - j)


def x_frag(par, j, half):
    base = FRAG_BASE + 8 * x_slot(par, j) + 4 * half
    return f"v[{base}:{base + 3}]"


def y_frag(i, half):
    base = FRAG_BASE + 8 * X_PAIRS + 8 * (i % Y_RING) + 4 * half
    return f"v[{base}:{base + 3}]"


def read_y(i, half):
    return f"ds_read_b128 {y_frag(i, half)}, {VW[half]}" + (f" offset:{2048 * i}" if i else "")


def read_x(par, j, half):
    return f"ds_read_b128 {x_frag(par, j, half)}, {VH[half]}" + (f" offset:{2048 * j}" if j else "")


def addr_ops(v, slot, row):
    return [f"v_add_u32 {v[0]}, %[{slot}], %[{row}]", f"v_xor_b32 {v[1]}, 64, {v[0]}"]


def pair_blocks():
    return [(i, j) for i in range(8) for j in (range(nb()) if i % 2 == 0 else range(nb() - 1, -1, -1))]


class Gaps:
    """What follows each MFMA of a step.  Two instructions fit behind an MFMA; `put` takes the first gap from `m` on that
    has room for a chunk (instructions that nothing may come between: SCC and VCC are shared)."""

    def __init__(self, n):
        self.at = [[] for _ in range(n)]

    def put(self, m, chunk, room=2):
        chunk = [chunk] if isinstance(chunk, str) else list(chunk)
        m = int(m)
        while self.at[m] and len(self.at[m]) + len(chunk) > room:
            m += 1
        self.at[m] += chunk
        return m

    def chain(self, m, chunks):
        for c in chunks:
            m = self.put(m, c) + 1
        return m


def next_slot_chunks(dst, slot, ring):
    ops = next_slot(dst, slot, ring)
    return [ops] if len(ops) == 1 else [[ops[0]], ops[1:3], [ops[3]]]


def copy_gaps(sync):
    """gaps of a step's copies, hidden then LM head, spread over the time from one sync to the next (beyond the step's last
    gap: in the next step)"""
    n, m = nb(), 16 * nb()
    first, h, end = sync + 2, m / 20, m + sync - 17
    w0 = first + n * h + 1
    at = [int(first + k * h) for k in range(n)] + [int(w0 + k * (end - w0) / 7) for k in range(8)]
    # M0 is written a gap ahead, in the same step, and its write changes SCC: not behind the loop's last comparison
    return [x if not m - 3 < x <= m else m - 3 if x < m - 1 else m + 1 for x in at]


def late_pieces():
    """of a step's eight LM-head copies, those that follow its sync (the others go ahead of the next one)"""
    return sum(m < 16 * nb() for m in copy_gaps(4 * nb() + 1)[nb():])


def pair_schedule(par):
    """(gaps, gap behind which the sync stands) of a step: reads, copies, scalars"""
    n, row, nxt = nb(), 2 * nb(), 1 - par
    gaps = Gaps(8 * row)
    sync = 2 * row + 1
    # this step's vocabulary blocks 2 and 3 ahead of the sync, 4..7 and the next step's 0 and 1 behind it; each once the
    # block four before it is done with
    for i, at in ((2, .4), (3, .9)):
        gaps.put(at * row, read_y(i, 0)), gaps.put(at * row + 2, read_y(i, 1))
    for k, x in enumerate(addr_ops(VH, "hrd", "rdh0")):      # the next step's hidden slot
        gaps.put(1.5 * row + 3 + k, x)
    hrot = [[f"s_xor_b32 %[hrd], %[hrd], {hex(h_slot())}"]] if h_slot() & (h_slot() - 1) == 0 else \
        [[f"s_add_u32 %[hrd], %[hrd], {hex(h_slot())}"], [f"s_cmp_ge_u32 %[hrd], {hex(h_ring())}", "s_cselect_b32 %[hrd], 0, %[hrd]"]]
    end = gaps.chain(1.3 * row, hrot)
    assert end <= 1.5 * row + 3
    gaps.at[sync] = ["sync"]
    # the hidden copies first, then the LM head's, the last of them ahead of the next sync
    copies = copy_gaps(sync)
    for k, m in enumerate(copies):
        setup, load = dma_split(k if k < n else k - n, hidden=k < n)
        m %= 8 * row
        assert gaps.put(m - 1, setup) == m - 1
        gaps.at[m].append(load)
    for i, at in ((4, 2.3), (5, 3.1), (6, 4.0), (7, 4.8)):
        gaps.put(at * row + 1, read_y(i, 0)), gaps.put(at * row + 3, read_y(i, 1))
    early = min(n, X_PAIRS - n)
    for k in range(2 * early):
        gaps.put(2.4 * row + 2 + k * 4.4 * row / (2 * early), read_x(nxt, k // 2, k % 2))
    wrot = [[f"s_add_u32 %[wrd], %[wrd], 0x8000"],
            [f"s_cmp_ge_u32 %[wrd], {hex(w_ring())}", "s_cselect_b32 %[wrd], 0, %[wrd]"]]
    end = gaps.chain(5.05 * row, wrot)
    for x in addr_ops(VW, "wrd", "rdw0"):
        end = gaps.put(end, x) + 1
    for i, at in ((0, max(end, 5.6 * row)), (1, 6.4 * row)):
        gaps.put(at, read_y(i, 0)), gaps.put(at + 2, read_y(i, 1))
    for k, j in enumerate(range(early, n)):                   # into the registers of block n - 1 - k, done with by then
        assert x_slot(nxt, j) == x_slot(par, n - 1 - k)
        gaps.put(7 * row + 4 * k + 1, read_x(nxt, j, 0)), gaps.put(7 * row + 4 * k + 3, read_x(nxt, j, 1))
    end = gaps.chain(copies[n - 1] + 1, [["s_add_u32 %[hk], %[hk], 1"], ["s_add_u32 s98, s98, 128", "s_addc_u32 s99, s99, 0"],
                                     ["s_cmp_eq_u32 %[hk], %[nk]", f"s_cselect_b32 vcc_lo, {NK128}, 0",
                                      "s_cselect_b32 %[hk], 0, %[hk]"],
                                     ["s_sub_u32 s98, s98, vcc_lo", "s_subb_u32 s99, s99, 0"]]
                     + next_slot_chunks("hdst", h_slot(), h_ring()))
    # past the unit's last K-tile the pointer stays
    wend = gaps.chain(copies[-1] % (8 * row) + 1,
                      [["s_add_u32 %[wk], %[wk], 1"],
                       ["s_cmp_eq_u32 %[wk], %[nk]", "s_cselect_b32 vcc_lo, %[wwrap], 128", "s_cselect_b32 %[wk], 0, %[wk]"],
                       ["s_add_u32 vcc_hi, %[g], %[wnext]"],
                       ["s_cmp_lt_u32 vcc_hi, %[total]", "s_cselect_b32 vcc_lo, vcc_lo, 0"],
                       ["s_add_u32 s96, s96, vcc_lo", "s_addc_u32 s97, s97, 0"]] + next_slot_chunks("wdst", 0x8000, w_ring()))
    # (the chains share VCC, and a pointer is on before its next copy)
    assert copies[-1] >= 8 * row and wend <= sync and end <= copies[-1]
    end = gaps.chain(max(end, 7 * row), [["s_add_u32 %[g], %[g], 1"], [f"s_add_u32 {KT}, {KT}, 1"]])
    end = max(end, *(m + 1 for m in copies if m < 8 * row))      # (an M0 write changes SCC)
    end = gaps.put(end, f"s_cmp_lt_u32 {KT}, %[nk]")
    return gaps.at, sync


def pair_waits():
    """wait[parity][m] = n: ahead of MFMA m of a step of this parity, lgkmcnt(n) (fragment reads return in order)"""
    wait = [{}, {}]
    issued, done, last = 0, 0, {}
    for par in range(2):
        for j in range(nb()):
            for h in range(2):
                issued += 1
                last[x_frag(0, j, h)] = issued
    for step in range(6):
        par = step % 2
        at, sync = pair_schedule(par)
        wait[par] = {}
        for m, (i, j) in enumerate(b for b in pair_blocks() for _ in range(2)):
            # for both halves of the block at once
            need = max(last.get(f, 0) for h in range(2) for f in (y_frag(i, h), x_frag(par, j, h)))
            if need > done:
                n = min(15, issued - need)
                wait[par][m] = n
                done = issued - n
            for x in at[m]:
                if x == "sync":
                    done = issued
                elif x.startswith("ds_read"):
                    issued += 1
                    last[x.split()[1].rstrip(",")] = issued
    return wait


def pair_step(par, wait):
    at, _ = pair_schedule(par)
    for m, (i, j) in enumerate(b for b in pair_blocks() for _ in range(2)):
        if m in wait[par]:
            e(f"s_waitcnt lgkmcnt({wait[par][m]})")
        e(f"v_mfma_f32_16x16x32_bf16 {acc_block(i, j)}, {y_frag(i, m % 2)}, {x_frag(par, j, m % 2)}, {acc_block(i, j)}")
        for x in at[m]:
            if x == "sync":
                # landed: all but the LM-head copies of the last step, the eight youngest
                e("s_waitcnt vmcnt(8) lgkmcnt(0)")
                e("s_barrier")
            else:
                e(x)


def build_pairs():
    e("s_mov_b32 s96, %[wsrc_lo]")
    e("s_mov_b32 s97, %[wsrc_hi]")
    e("s_mov_b32 s98, %[hsrc_lo]")
    e("s_mov_b32 s99, %[hsrc_hi]")
    e(f"s_add_u32 {NK128}, %[hwrap], 128")
    e(f"s_mov_b32 {KT}, 0")
    for x in addr_ops(VW, "wrd", "rdw0") + addr_ops(VH, "hrd", "rdh0"):
        e(x)
    for h in range(2):
        e(read_y(0, h))
    for j in range(nb()):
        for h in range(2):
            e(read_x(0, j, h))
    for h in range(2):
        e(read_y(1, h))
    for i in range(32 * nb()):
        e(f"v_accvgpr_write_b32 a{i}, 0")
    e("s_nop 7")
    e("s_waitcnt lgkmcnt(0)")
    wait = pair_waits()
    top, out = label("steady"), label("out")
    e(f"{top}:")
    pair_step(0, wait)
    e(f"s_cbranch_scc0 {out}")
    pair_step(1, wait)
    e(f"s_cbranch_scc1 {top}")
    e(f"{out}:")
    e("s_waitcnt lgkmcnt(0)")
    e("s_nop 15")
    e("s_nop 15")
    e("s_mov_b32 %[wsrc_lo], s96")
    e("s_mov_b32 %[wsrc_hi], s97")
    e("s_mov_b32 %[hsrc_lo], s98")
    e("s_mov_b32 %[hsrc_hi], s99")


def write_statement(f, blocks, sample):
    SHAPE["nb"] = blocks
    lines.clear()
    uid[0] = 2000 if sample else 1000
    if sample:
        build_tile_sample()
        outs = []
        for tb in range(blocks):
            outs += [f'[m{tb}] "=&v"(tile_m[{tb}])', f'[s{tb}] "=&v"(tile_s[{tb}])', f'[i{tb}] "+v"(run_i[{tb}])',
                     f'[ym{tb}] "+v"(run_ym[{tb}])', f'[xa{tb}] "+v"(run_xa[{tb}])']
    else:
        build_tile()
        outs = []
        for tb in range(blocks):
            outs += [f'[m{tb}] "=&v"(tile_m[{tb}])', f'[s{tb}] "=&v"(tile_s[{tb}])', f'[i{tb}] "=&v"(tile_i[{tb}])']
    for name in ("wsrc_lo", "wsrc_hi", "hsrc_lo", "hsrc_hi", "wrd", "hrd", "wdst", "hdst", "wk", "hk", "g"):
        outs.append(f'[{name}] "+s"(st_{name})')
    outs.append('[vt0] "=&v"(addr_tmp0)')
    outs.append('[vt1] "=&v"(addr_tmp1)')
    ins = []
    if pairs():
        outs += ['[vt2] "=&v"(addr_tmp2)', '[vt3] "=&v"(addr_tmp3)']
        ins.append('[wnext] "s"(st_wnext)')
    for k in range(1 if pairs() else 2):
        ins.append(f'[rdw{k}] "v"(rdw[{k}])')
        ins.append(f'[rdh{k}] "v"(rdh[{k}])')
    for i in range(8):
        ins.append(f'[woff{i}] "v"(woff[{i}])')
    for i in range(blocks):
        ins.append(f'[hoff{i}] "v"(hoff[{i}])')
    for name in ("total", "nk", "wwrap", "hwrap"):
        ins.append(f'[{name}] "s"(st_{name})')
    clob = ['"s94"', '"s95"', '"s96"', '"s97"', '"s98"', '"s99"', '"vcc"', '"scc"', '"m0"', '"memory"']
    ins += ['[vb] "v"(vb)', '[first] "s"(st_first)', '[nt] "n"(STREAM ? 1 : 0)']
    clob = [f'"a{i}"' for i in range(32 * blocks)] + [f'"s{i}"' for i in range(88, 94)] + clob
    if sample:
        ins += [f'[pos{tb}] "v"(pos[{tb}])' for tb in range(blocks)]
        ins += ['[rb] "s"(row_best)', '[rl] "s"(last_row)']
        ins += ['[seed_lo] "s"(seed_lo)', '[seed_hi] "s"(seed_hi)']
        clob = [f'"s{i}"' for i in range(66, KEY1_BASE + 10)] + clob
        ins += ['[pm0] "s"(philox_m0)', '[pm1] "s"(philox_m1)', '[itl] "s"(inv_tau_log2e)', '[tau] "s"(tau_s)']
    clob = [f'"v{i}"' for i in range(FRAG_BASE, FRAG_BASE + 128)] + clob
    f.write(f"if constexpr (NB == {blocks}) {{\nasm volatile(\n")
    for ln in lines:
        if ln.startswith("global_load_lds_dwordx4 %[woff"):     # the LM head, as the kernel's launch streams it or not
            f.write(f'    ".if %[nt]\\n{ln} nt\\n.else\\n{ln}\\n.endif\\n"\n')
        else:
            f.write(f'    "{ln}\\n"\n')
    f.write("    : " + ",\n      ".join(outs) + "\n")
    f.write("    : " + ",\n      ".join(ins) + "\n")
    f.write("    : " + ", ".join(clob) + ");\n}\n")


def write_pieces(f):
    """what the kernel's prologue has to know of the K-loop: the first width in pair order, and that loop's late_pieces"""
    pieces = [0] * 9
    for blocks in range(PAIRS_FROM, 9):
        SHAPE["nb"] = blocks
        pieces[blocks] = late_pieces()
    f.write("// GENERATED by gen_w4_loop.py -- do not edit.\n"
            f"constexpr int kW4PairsFrom = {PAIRS_FROM};\n"
            f"constexpr int kW4Take = (int){hex(TAKE)}u;\n"
            f"constexpr int w4_late_pieces(int nb) {{\n  constexpr int pieces[9] = {{{', '.join(map(str, pieces))}}};\n"
            "  return pieces[nb];\n}\n")


def main(folder):
    for name, sample in (("mosaic_w4_tile.inc", False), ("mosaic_w4_tile_sample.inc", True)):
        with open(os.path.join(folder, name), "w") as f:
            f.write("// GENERATED by gen_w4_loop.py -- do not edit.  One vocabulary tile of the "
                    f"{'sampling' if sample else 'greedy'} 4-wave kernel, K-loop and vocabulary reduction, per width.\n")
            for blocks in range(1, 9):
                write_statement(f, blocks, sample)
    with open(os.path.join(folder, "mosaic_w4_pieces.inc"), "w") as f:
        write_pieces(f)


if __name__ == "__main__":
    main(sys.argv[1] if len(sys.argv) > 1 else os.path.dirname(os.path.abspath(__file__)))
