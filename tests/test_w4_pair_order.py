"""The K-loop in pair order (both K-halves of a block's products back to back), the one of the wide row tiles, interpreted
on the CPU for an even and an odd wave side by side, which copy different K-tiles of the LM head in one step.

LDS is modelled by regions: the vocabulary blocks 0..3 and 4..7 of an LM-head slot, filled by the even and the odd waves,
and a hidden slot, filled by all.  A copy may only go to a region that no wave has read since the last barrier; a region is
readable again once every wave that fills it has waited for its copies (vmcnt, in issue order) and met the others at a
barrier.  A fragment is usable once an lgkmcnt wait covers its read (in issue order).  Every product must find the
vocabulary block, token block, K-tile and K-half it stands for, first half then second half of a block."""
import os
import re
import subprocess

import pytest

import test_w4_loop_protocol as protocol
from test_w4_loop_protocol import H_BASE, MASK32, W_BASE, gen

WIDTHS = range(gen.PAIRS_FROM, 9)
LATE = {}
for width in WIDTHS:
    gen.SHAPE["nb"] = width
    LATE[width] = gen.late_pieces()


def listing(nb, sample=False):
    return protocol.listing(nb, sample)[0]


class Lds:
    def __init__(self):
        self.holds, self.pending, self.reads = {}, {}, set()

    def barrier(self, waves):
        assert not any(w.lgkm for w in waves), "barrier with fragment reads in flight"
        for region, parts in list(self.pending.items()):
            fillers = {0, 1} if region[0] == "H" else {0 if region[2] == "lo" else 1}
            if set(parts) == fillers and all(landed for _, landed, _ in parts.values()):
                ids = {ident for ident, _, _ in parts.values()}
                assert len(ids) == 1
                self.holds[region] = ids.pop()
                del self.pending[region]
        self.reads.clear()


class PairWave(protocol.Sim):
    """One wave's stream up to its next barrier at a time (the base class's instruction set, its own events)."""

    def __init__(self, lines, nb, nk, ntile, ragged_rows, odd, lds):
        super().__init__(lines, nb, nk, ntile, ragged_rows)
        self.odd, self.lds = odd, lds
        self.lgkm, self.frags, self.used, self.copied = [], {}, {}, {"W": 0, "H": 0}
        self.n, self.blocks = 0, set()

    def w_region(self, slot):
        return ("W", slot, "hi" if self.odd else "lo")

    def prologue(self):
        lead = 2 if self.odd else 3
        for op, g in ([("W", 0), ("H", 0)] + ([] if self.odd else [("W", 1)]) + [("H", 1), ("W", lead - 1)]):
            if op == "W" and g == lead - 1:                      # the first pieces; the first step copies the others
                self.lds.pending.setdefault(self.w_region(g % 3), {})[int(self.odd)] = (g, False, LATE[self.nb])
                self.vm_queue += [self.w_region(g % 3)] * LATE[self.nb] * (self.total >= 3)
            elif g < self.total:
                region = ("H", g % 2) if op == "H" else self.w_region(g % 3)
                if g == 0 or self.total < 3:                     # the kernel waits for all of a short unit's copies
                    self.lds.holds[region] = g
                else:
                    self.lds.pending.setdefault(region, {})[int(self.odd)] = (g, False, self.nb if op == "H" else 8)
                    self.vm_queue += [region] * (self.nb if op == "H" else 8)
        self.copied = {"W": lead - 1, "H": 2}
        w, h = self.wptr(min(lead - 1, self.total - 1)), H_BASE + 2 % self.nk * 128
        self.reg.update({
            "%[wsrc_lo]": w & MASK32, "%[wsrc_hi]": w >> 32, "%[hsrc_lo]": h & MASK32, "%[hsrc_hi]": h >> 32,
            "%[wrd]": 0, "%[hrd]": 0, "%[wdst]": (lead - 1) % 3 * 0x8000 + 1024 * self.turn, "%[hdst]": 0, "%[wk]": min(lead - 1, self.total - 1) % self.nk,
            "%[hk]": 2 % self.nk, "%[g]": 0, "%[total]": self.total, "%[nk]": self.nk, "%[hwrap]": (self.nk - 1) * 128,
            "%[wnext]": lead, "%[rdw0]": 0, "%[rdh0]": 0x18000})

    def begin(self, n):
        rows = self.ragged_rows if self.ragged_rows and n + 2 == self.ntile else 256
        self.reg["%[wwrap]"] = (rows * self.nk * 128 - (self.nk - 1) * 128) & MASK32
        self.pc, self.ran = 0, 0
        self.frags.clear()
        self.used.clear()
        self.started.clear()

    def copy(self, op, offset):
        m0, off = self.reg["m0"], None
        if op == "W":
            ident, region, slot = self.copied["W"], self.w_region(self.copied["W"] % 3), m0 // 0x8000
            source = self.wptr(min(ident, self.total - 1))       # past the end the last tile once more, which nobody reads
            assert (self.reg["s96"] | self.reg["s97"] << 32) == source and slot == ident % 3
            off, pieces = m0 % 0x8000, 8
        else:
            ident, region = self.copied["H"], ("H", self.copied["H"] % 2)
            assert (self.reg["s98"] | self.reg["s99"] << 32) == H_BASE + ident % self.nk * 128
            slot, off = divmod(m0 - 0x18000, self.nb * 0x1000)
            assert slot == ident % 2
            pieces = self.nb
        assert region not in self.lds.reads, f"copy into {region}, which a wave may still be reading"
        parts = self.lds.pending.setdefault(region, {})
        done = parts[int(self.odd)][2] if int(self.odd) in parts else 0
        piece = self.source_piece(op, offset)
        assert off == 1024 * piece, f"piece {piece} of a tile goes to byte {off} of the slot, not to its own KiB"
        assert done < pieces and piece == (done ^ self.turn if op == "W" else done), "every piece once, in the unit's order"
        parts[int(self.odd)] = (ident, False, done + 1)
        self.lds.holds.pop(region, None)
        self.vm_queue.append(region)
        if done + 1 == pieces:
            self.copied[op] += 1

    def wait_vm(self, n):
        while len(self.vm_queue) > n:
            region = self.vm_queue.pop(0)
            if region not in self.vm_queue:
                ident, _, pieces = self.lds.pending[region][int(self.odd)]
                if pieces == (self.nb if region[0] == "H" else 8):
                    self.lds.pending[region][int(self.odd)] = (ident, True, pieces)

    def ds_read(self, dst, addr_reg, offset):
        addr = self.reg[addr_reg] + offset
        if addr < 0x18000:
            slot, rest = divmod(addr, 0x8000)
            block = rest // 2048
            region, op = ("W", slot, "lo" if block < 4 else "hi"), "W"
        else:
            slot, rest = divmod(addr - 0x18000, self.nb * 0x1000)
            block = rest // 2048
            region, op = ("H", slot), "H"
            assert slot < 2 and block < self.nb
        assert rest % 2048 in (0, 64)
        first = int(re.fullmatch(r"v\[(\d+):\d+\]", dst).group(1))
        assert (first >= 208) == (op == "W") and 112 <= first <= 236 and first % 4 == 0
        assert self.n - self.used.get(dst, -9) >= 2, f"{dst} overwritten right behind the product that uses it"
        # a read of a step that does not come may find anything, but never a slot that a copy is on its way into
        assert region not in self.lds.pending, f"read of {region} with a copy under way"
        self.lds.reads.add(region)
        self.lgkm.append(dst)
        self.frags[dst] = (op, self.lds.holds.get(region), block, rest % 2048 // 64)

    def mfma(self, a, b, dst, src_c):
        step, m = divmod(self.n, 16 * self.nb)
        g, half = step, m % 2
        base, top = (int(x) for x in re.fullmatch(r"a\[(\d+):(\d+)\]", dst).groups())
        assert top == base + 3 and base % 4 == 0 and src_c == dst and set(range(base, top + 1)) <= self.started
        i, j = divmod(base // 4, self.nb)
        if half == 0:
            self.block = (i, j)
            assert (g, i, j) not in self.blocks
            self.blocks.add((g, i, j))
        assert self.block == (i, j)
        assert a not in self.lgkm and b not in self.lgkm, "fragment used before its wait"
        assert self.frags[a] == ("W", g, i, half), (self.frags[a], g, i, half)
        assert self.frags[b] == ("H", g, j, half), (self.frags[b], g, j, half)
        self.used[a] = self.used[b] = self.n
        self.n += 1

    def until_barrier(self):
        """True: stopped behind a barrier's issue; False: the statement has ended"""
        while self.pc < len(self.prog):
            self.ran += 1
            assert self.ran < 400000, "the loop does not terminate"
            ins = self.prog[self.pc]
            self.pc += 1
            op, _, rest = ins.partition(" ")
            args = [x.strip() for x in rest.split(",")] if rest else []
            if op == "s_barrier":
                return True
            if op == "v_mfma_f32_16x16x32_bf16":
                self.mfma(args[1], args[2], args[0], args[3])
            elif op == "v_accvgpr_write_b32":
                self.started.add(int(args[0][1:]))
            elif op == "ds_read_b128":
                m = re.fullmatch(r"(\S+)(?: offset:(\d+))?", args[1])
                self.ds_read(args[0], m.group(1), int(m.group(2) or 0))
            elif op == "global_load_lds_dwordx4":
                assert not protocol.writes_m0(self.prog[self.pc - 2]), "no instruction between the write of M0 and the load"
                self.copy("W" if args[1].split()[0] == "s[96:97]" else "H", args[0])
            elif op == "v_add_u32":
                self.set(args[0], self.val(args[1]) + self.val(args[2]))
            elif op == "v_xor_b32":
                self.set(args[0], self.val(args[1]) ^ self.val(args[2]))
            elif op == "s_waitcnt":
                for counter, n in re.findall(r"(vmcnt|lgkmcnt)\((\d+)\)", rest):
                    assert int(n) <= (63 if counter == "vmcnt" else 15)
                    if counter == "vmcnt":
                        self.wait_vm(int(n))
                    else:
                        del self.lgkm[:max(0, len(self.lgkm) - int(n))]
            elif op == "s_nop":
                pass
            elif op == "s_mov_b32":
                self.set(args[0], self.val(args[1]))
            elif op in ("s_add_u32", "s_addc_u32"):
                r = self.val(args[1]) + self.val(args[2]) + (self.scc if op == "s_addc_u32" else 0)
                self.set(args[0], r)
                self.scc = 1 if r > MASK32 else 0
            elif op in ("s_sub_u32", "s_subb_u32"):
                r = self.val(args[1]) - self.val(args[2]) - (self.scc if op == "s_subb_u32" else 0)
                self.set(args[0], r)
                self.scc = 1 if r < 0 else 0
            elif op == "s_xor_b32":
                self.set(args[0], self.val(args[1]) ^ self.val(args[2]))
                self.scc = int(self.val(args[0]) != 0)
            elif op == "s_cselect_b32":
                self.set(args[0], self.val(args[1]) if self.scc else self.val(args[2]))
            elif op.startswith("s_cmp_"):
                x, y = self.val(args[0]), self.val(args[1])
                self.scc = int({"s_cmp_lt_u32": x < y, "s_cmp_ge_u32": x >= y, "s_cmp_eq_u32": x == y}[op])
            elif op == "s_branch" or op == f"s_cbranch_scc{self.scc}":
                self.pc = self.labels[args[0]]
            else:
                assert op in ("s_cbranch_scc0", "s_cbranch_scc1"), f"instruction the checker does not know: {ins}"
        assert not self.lgkm
        return False


def run(lines, nb, nk, ntile, ragged=0, turn=0):
    lds = Lds()
    waves = [PairWave(lines, nb, nk, ntile, ragged, odd, lds) for odd in (False, True)]
    for w in waves:
        w.turn = turn
        w.prologue()
    for n in range(ntile):
        for w in waves:
            w.begin(n)
        while True:
            at_barrier = [w.until_barrier() for w in waves]
            assert at_barrier[0] == at_barrier[1], "the waves disagree about a barrier"
            if not at_barrier[0]:
                break
            lds.barrier(waves)
    total = nk * ntile
    for w in waves:
        assert w.n == 16 * nb * total and len(w.blocks) == 8 * nb * total and w.reg["%[g]"] == total
        assert w.started == set(range(32 * nb))
        assert w.copied == {"W": total + (1 if w.odd else 2), "H": total + 2}      # one of each a step


SHAPES = [(1, 1, 0), (1, 5, 0), (2, 1, 0), (2, 3, 0), (3, 1, 0), (3, 4, 0), (4, 2, 0), (5, 31, 0), (8, 2, 0), (56, 2, 0),
          (64, 1, 0), (5, 1, 7), (5, 2, 1), (5, 4, 255), (6, 3, 128), (9, 2, 77)]


@pytest.mark.parametrize("sample", [False, True])
@pytest.mark.parametrize("nb", WIDTHS)
def test_pair_order_protocol(nb, sample):
    loop = listing(nb, sample)
    for nk, ntile, ragged in SHAPES:
        run(loop, nb, nk, ntile, ragged)


@pytest.mark.parametrize("nb", WIDTHS)
@pytest.mark.parametrize("mistake", ["no vmcnt", "no lgkmcnt", "late vmcnt", "barrier early", "one lead for all", "W load behind M0",
                                     "H load behind M0"])
def test_planted_mistakes_are_caught(nb, mistake, monkeypatch):
    """Planted in a copy of the listing, or in the checker's glue."""
    loop = listing(nb)
    if mistake == "no vmcnt":
        loop = [re.sub(r"vmcnt\(\d+\) ", "", ln) for ln in loop]
    elif mistake == "no lgkmcnt":
        loop = [ln for ln in loop if not re.fullmatch(r"s_waitcnt lgkmcnt\(([1-9]|1\d)\)", ln)]
    elif mistake == "late vmcnt":
        loop = [re.sub(r"vmcnt\(8\)", f"vmcnt({8 + nb})", ln) for ln in loop]
    elif mistake.endswith("M0"):
        loop = protocol.without_wait_state(loop, "%[wdst]" if mistake[0] == "W" else "%[hdst]")
    elif mistake == "barrier early":
        at = next(i for i, ln in enumerate(loop) if ln == "s_barrier")
        first = next(i for i, ln in enumerate(loop) if ln.startswith("v_mfma"))
        wait = loop[at - 1]
        loop = loop[:first + 1] + [wait, "s_barrier"] + loop[first + 1:at - 1] + loop[at + 1:]
    else:
        monkeypatch.setattr(PairWave, "w_region", lambda self, slot: ("W", slot, "hi"))
    with pytest.raises(AssertionError, match="M0" if mistake.endswith("M0") else None):
        run(loop, nb, 6, 3)


@pytest.mark.parametrize("nb", WIDTHS)
def test_steady_steps_keep_every_gap_short(nb):
    loop = listing(nb)
    start = next(i for i, ln in enumerate(loop) if ln.startswith("Lsteady"))
    end = next(i for i, ln in enumerate(loop) if ln.startswith("Lout"))
    gap, longest = 0, 0
    for ln in loop[start + 1:end - 1]:
        if ln.startswith("v_mfma"):
            longest, gap = max(longest, gap), 0
        else:
            gap += 1
    assert longest <= 4, longest


def test_the_kernel_learns_the_first_width_in_pair_order(tmp_path, monkeypatch):
    """The rings' prologue is the kernel's, the loop the generator's: from which width on, and how many of a step's copies
    follow its sync, is written once and read from the generated header, whatever the first width is."""
    for first in (gen.PAIRS_FROM, 6):
        monkeypatch.setattr(gen, "PAIRS_FROM", first)
        with open(tmp_path / "pieces.inc", "w") as f:
            gen.write_pieces(f)
        late = {}
        for nb in range(first, 9):
            gen.SHAPE["nb"] = nb
            late[nb] = gen.late_pieces()
        gen.SHAPE["nb"] = 8
        checks = "".join(f"static_assert(w4_late_pieces({nb}) == {late.get(nb, 0)}, \"\");\n" for nb in range(1, 9))
        (tmp_path / "check.cpp").write_text(f'#include "pieces.inc"\nstatic_assert(kW4PairsFrom == {first}, "");\n{checks}')
        subprocess.run(["g++", "-std=c++17", "-fsyntax-only", str(tmp_path / "check.cpp")], check=True)
    kernel = open(os.path.join(os.path.dirname(protocol.GEN), "mosaic_logits.hip")).read()
    assert "kPairs = NB >= kW4PairsFrom;" in kernel
