"""The generated K-loop of the 4-wave kernel's narrow row tiles (32 to 128 tokens, one K-half after the other; the wide ones
are test_w4_pair_order.py's), interpreted on the CPU (no GPU): the scalar book-keeping is executed
instruction by instruction and every copy, LDS read, wait, barrier and MFMA is checked against the ring protocol.

What is proved for each width and (K-tiles per vocabulary tile, vocabulary tiles per unit) tried:
  * every direct-to-LDS copy reads a tile that exists (its source pointer decodes to a step below the total: no
    out-of-bounds global read) and each tile is copied exactly once, in order;
  * a copy never targets a slot that any wave may still read (no LDS read of that slot between the two barriers
    around the copy), and a slot is never read while a copy into it is not yet published;
  * a copy is "published" only by a vmcnt wait that covers it followed by a barrier; every LDS read finds the tile
    and K-half it expects;
  * every MFMA group multiplies fragments that were read, waited for (lgkmcnt) and belong to its step and K-half;
  * fragment registers are not overwritten while the group that uses them is still issuing.
Waves run the same instruction stream and meet at every barrier, so one wave's stream plus "anything between two
barriers may overlap across waves" covers the workgroup.
"""
import importlib.util
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
GEN = os.path.join(ROOT, "paper_2601_06562_amd", "csrc", "gen_w4_loop.py")

SLOT = 0x8000                                          # of the LM head; a hidden slot has 4 KiB per token block
W_BASE, H_BASE = 0x10_0000_0000, 0x20_0000_0000       # synthetic device addresses
MASK32 = 0xFFFFFFFF

spec = importlib.util.spec_from_file_location("gen_w4_loop", GEN)
gen = importlib.util.module_from_spec(spec)
spec.loader.exec_module(gen)
WIDTHS = range(1, gen.PAIRS_FROM)


def listing(nb, sample=False):
    """A width's statement as it is built in: its K-loop, the ragged tile's part, the reduction."""
    gen.SHAPE["nb"] = nb
    gen.lines.clear()
    gen.uid[0] = 0
    gen.build_tile_sample() if sample else gen.build_tile()
    out = [ln.strip() for ln in gen.lines]
    gen.lines.clear()
    gen.SHAPE["nb"] = 8
    cut = out.index("s_cmp_eq_u32 %[first], 0")
    end = next(i for i in range(cut, len(out)) if out[i].startswith("Lwhole")) + 1
    return out[:cut], out[cut:end], out[end:]


def writes_m0(ins):
    """A direct-to-LDS load needs an instruction between the write of M0, by whatever operation, and itself."""
    return re.match(r"s_\w+ m0,", ins) is not None


def without_wait_state(lines, base):
    """A planted mistake: the first write of M0 from `base` right ahead of its load."""
    at = next(i for i, ln in enumerate(lines) if writes_m0(ln) and base in ln)
    load = next(i for i in range(at, len(lines)) if lines[i].startswith("global_load_lds"))
    return lines[:at] + lines[at + 1:load] + [lines[at]] + lines[load:]


class Sim:
    turn = 0                                     # of this unit's LM-head copies: copy i brings piece i ^ turn to its place

    def __init__(self, lines, nb, nk, ntile, ragged_rows=0):
        self.nb, self.nk, self.ntile, self.total = nb, nk, ntile, nk * ntile
        self.ragged_rows = ragged_rows           # rows from the last tile but one to the last one, 0: 256 as elsewhere
        self.nh = 3 if nb <= 2 else 2
        self.nw = self.nh + 1
        assert self.nw * SLOT + self.nh * nb * 0x1000 <= 160 * 1024
        self.prog = []
        self.labels = {}
        for ln in lines:
            ln = ln.strip()
            if ln.endswith(":"):
                self.labels[ln[:-1]] = len(self.prog)
            elif ln:
                self.prog.append(ln)
        self.reg = {}
        self.scc = 0
        # ring state: what each slot holds (published), what is in flight, who read it since the last barrier
        self.published = {}            # slot -> tile id (W: step g, H: k index)
        self.unpublished = {}          # slot -> tile id, copy issued but not yet covered by wait + barrier
        self.landed = set()            # slots whose in-flight copy a vmcnt wait has covered (await the barrier)
        self.vm_queue = []             # destination slots of the outstanding copy instructions, in issue order
        self.reads_this_interval = set()
        self.copies_this_interval = set()
        self.next_w_copy, self.next_h_copy = 0, 0
        self.frag = {}                 # fragment register name -> (operand, tile id, khalf, complete?)
        self.mfma_count = 0
        self.frag_last_group = {}      # fragment register -> last MFMA group that used it
        self.copy_parts = {}           # slot -> pieces issued for the current copy (of 8, of hidden rows nb, per wave)
        self.started = set()           # accumulator registers (by number) started in the current statement

    # ---- operand access
    def val(self, tok):
        tok = tok.strip()
        if re.fullmatch(r"-?\d+", tok):
            return int(tok) & MASK32
        if tok.startswith("0x"):
            return int(tok, 16) & MASK32
        return self.reg[tok]

    def set(self, tok, v):
        self.reg[tok.strip()] = v & MASK32

    # ---- events
    def slot_of(self, addr):
        ring = self.nw * SLOT
        slot = addr // SLOT if addr < ring else self.nw + (addr - ring) // (self.nb * 0x1000)
        assert slot < self.nw + self.nh
        return slot

    def offset_in(self, addr):
        ring = self.nw * SLOT
        return addr % SLOT if addr < ring else (addr - ring) % (self.nb * 0x1000)

    def wptr(self, g):
        tile = g // self.nk
        rows = tile * 256
        if self.ragged_rows and tile == self.ntile - 1 and tile > 0:
            rows += self.ragged_rows - 256
        return W_BASE + rows * (self.nk * 128) + (g % self.nk) * 128

    def source_piece(self, operand, offset):
        """The piece of a tile that a copy's offsets stand for, which the kernel makes: %[woff i] is piece i ^ turn."""
        i = int(re.fullmatch(r"%\[[wh]off(\d)\]", offset).group(1))
        return i ^ self.turn if operand == "W" else i

    def copy(self, operand, offset):
        m0 = self.reg["m0"]
        slot = self.slot_of(m0)
        assert slot not in self.reads_this_interval, f"copy into slot {slot} that a wave may still be reading"
        if operand == "W":
            ident, pieces = self.next_w_copy, 8
            assert ident < self.total, f"W copy of step {ident} beyond the {self.total} steps (out-of-bounds read)"
            assert (self.reg["s96"] | self.reg["s97"] << 32) == self.wptr(ident)
            assert slot == ident % self.nw
        else:
            off = (self.reg["s98"] | self.reg["s99"] << 32) - H_BASE
            ident, pieces = off // 128, self.nb
            assert off % 128 == 0 and 0 <= ident < self.nk, f"H pointer {off} outside the row"
            assert self.next_h_copy < self.total, "hidden copy past the last step"
            assert ident == self.next_h_copy % self.nk and slot - self.nw == self.next_h_copy % self.nh
        parts = self.copy_parts.get(slot, 0)
        if parts == 0:
            assert slot not in self.unpublished, f"second copy into slot {slot} before the first was published"
            self.unpublished[slot] = ident
            self.copies_this_interval.add(slot)
        assert self.unpublished[slot] == ident
        place, piece = self.offset_in(m0), self.source_piece(operand, offset)
        assert place == 1024 * piece, f"piece {piece} of a tile goes to byte {place} of the slot, not to its own KiB"
        assert piece == (parts ^ self.turn if operand == "W" else parts), "every piece once, in the unit's order"
        self.copy_parts[slot] = (parts + 1) % pieces
        self.vm_queue.append(slot)
        if self.copy_parts[slot] == 0:
            if operand == "W":
                self.next_w_copy += 1
            else:
                self.next_h_copy += 1

    def wait_vm(self, n):
        while len(self.vm_queue) > n:
            slot = self.vm_queue.pop(0)
            if slot not in self.vm_queue and self.copy_parts.get(slot, 0) == 0:
                self.landed.add(slot)

    def barrier(self):
        for slot in list(self.landed):
            self.published[slot] = self.unpublished.pop(slot)
        self.landed.clear()
        self.reads_this_interval.clear()
        self.copies_this_interval.clear()

    def ds_read(self, dst, addr_reg, offset):
        base = self.reg[addr_reg]
        slot = self.slot_of(base + offset)
        khalf = 1 if self.offset_in(base) % 128 == 64 else 0
        operand = "W" if slot < self.nw else "H"
        assert self.slot_of(base) == slot
        assert (operand == "W") == (addr_reg == "%[vt0]"), "LM-head fragments come from the LM-head ring"
        first = int(re.fullmatch(r"v\[(\d+):\d+\]", dst).group(1))     # LM-head tuples first in each buffer of 16
        assert (first - 112) // 4 % 16 == offset // 2048 + (0 if operand == "W" else 8)
        assert slot not in self.unpublished, f"read of slot {slot} while a copy into it is not published"
        assert slot in self.published, f"read of slot {slot} that holds nothing"
        assert slot not in self.copies_this_interval
        self.reads_this_interval.add(slot)
        group, within = divmod(self.mfma_count, 8 * self.nb)
        assert self.frag_last_group.get(dst, -1) < group or within == 0, f"{dst} overwritten while its group is still issuing"
        self.frag[dst] = (operand, self.published[slot], khalf, False)

    def wait_lgkm(self):
        for k, f in self.frag.items():
            self.frag[k] = (f[0], f[1], f[2], True)

    def mfma(self, a, b, dst, src_c):
        m = re.fullmatch(r"a\[(\d+):(\d+)\]", dst)
        regs = set(range(int(m.group(1)), int(m.group(2)) + 1))
        assert src_c == dst and regs <= self.started, f"accumulation into {dst}, which was never started"
        group = self.mfma_count // (8 * self.nb)
        g, h = divmod(group, 2)
        for name, operand in ((a, "W"), (b, "H")):
            assert name in self.frag, f"{name} used before it was read"
            f = self.frag[name]
            assert f[3], f"{name} used before the lgkmcnt wait"
            want = g if operand == "W" else g % self.nk
            assert f[0] == operand and f[1] == want and f[2] == h, \
                f"step {g} half {h}: {name} holds {f}, wanted {operand} {want}"
            self.frag_last_group[name] = group
        self.mfma_count += 1

    # ---- the glue around the statement, as the kernel's C++ does it
    def prologue(self):
        NW, NH = self.nw, self.nh
        # the kernel issues W0, H0, W1 and what else the rings hold, waits for the first two only, then meets at a barrier
        self.published[0] = 0
        self.published[NW] = 0
        for g in range(1, min(NW, self.total)):
            self.unpublished[g] = g
            self.vm_queue += [g] * 8
        for g in range(1, min(NH, self.total)):
            self.unpublished[NW + g] = g % self.nk
            self.vm_queue += [NW + g] * self.nb
        self.next_w_copy, self.next_h_copy = NW, NH
        w, h = self.wptr(NW), H_BASE + (NH % self.nk) * 128
        self.reg.update({
            "%[wsrc_lo]": w & MASK32, "%[wsrc_hi]": w >> 32, "%[hsrc_lo]": h & MASK32, "%[hsrc_hi]": h >> 32,
            "%[wrd]": 0, "%[hrd]": 0, "%[wdst]": 1024 * self.turn, "%[hdst]": 0, "%[wk]": NW % self.nk, "%[hk]": NH % self.nk,
            "%[g]": 0, "%[total]": self.total, "%[nk]": self.nk,
            "%[hwrap]": (self.nk - 1) * 128,
            "%[rdw0]": 0, "%[rdw1]": 64, "%[rdh0]": NW * SLOT, "%[rdh1]": NW * SLOT + 64,
        })

    def run_tiles(self):
        for n in range(self.ntile):              # the kernel hands every statement its step into the next tile
            rows = self.ragged_rows if self.ragged_rows and n + 2 == self.ntile else 256
            self.reg["%[wwrap]"] = (rows * self.nk * 128 - (self.nk - 1) * 128) & MASK32
            self.run_statement()

    def run_statement(self):
        self.frag.clear()                 # fragment registers do not survive between statements
        self.frag_last_group.clear()
        self.started.clear()              # nor do accumulators the statement addresses by number
        pc, steps = 0, 0
        while pc < len(self.prog):
            steps += 1
            assert steps < 200000, "the loop does not terminate"
            ins = self.prog[pc]
            pc += 1
            op, _, rest = ins.partition(" ")
            args = [a.strip() for a in rest.split(",")] if rest else []
            if op == "v_mfma_f32_16x16x32_bf16":
                self.mfma(args[1], args[2], args[0], args[3])
            elif op == "v_accvgpr_write_b32":
                assert args[1] == "0" and self.mfma_count % (16 * self.nb) == 0
                self.started.add(int(args[0][1:]))
            elif op == "ds_read_b128":
                m = re.fullmatch(r"(\S+)(?: offset:(\d+))?", args[1])
                self.ds_read(args[0], m.group(1), int(m.group(2) or 0))
            elif op == "global_load_lds_dwordx4":
                assert not writes_m0(self.prog[pc - 2]), "no instruction between the write of M0 and the load that reads it"
                self.copy("W" if args[1] == "s[96:97]" else "H", args[0])
            elif op == "v_add_u32":
                self.set(args[0], self.val(args[1]) + self.val(args[2]))
            elif op == "s_waitcnt":
                counters = re.findall(r"(vmcnt|lgkmcnt)\((\d+)\)", rest)
                assert counters and " ".join(f"{c}({n})" for c, n in counters) == rest.strip()
                for counter, n in counters:          # one instruction may wait on both counters
                    if counter == "vmcnt":
                        self.wait_vm(int(n))
                    else:
                        assert n == "0"
                        self.wait_lgkm()
            elif op == "s_barrier":
                assert all(f[3] for f in self.frag.values()), "barrier with LDS reads still in flight"
                self.barrier()
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
            elif op in ("s_xor_b32", "s_and_b32"):
                r = self.val(args[1]) ^ self.val(args[2]) if op == "s_xor_b32" else self.val(args[1]) & self.val(args[2])
                self.set(args[0], r)
                self.scc = 1 if r != 0 else 0
            elif op == "s_cselect_b32":
                self.set(args[0], self.val(args[1]) if self.scc else self.val(args[2]))
            elif op.startswith("s_cmp_"):
                a, b = self.val(args[0]), self.val(args[1])
                self.scc = int({"s_cmp_lt_u32": a < b, "s_cmp_ge_u32": a >= b, "s_cmp_eq_u32": a == b}[op])
            elif op == "s_branch":
                pc = self.labels[args[0]]
            elif op == "s_cbranch_scc0":
                if not self.scc:
                    pc = self.labels[args[0]]
            elif op == "s_cbranch_scc1":
                if self.scc:
                    pc = self.labels[args[0]]
            else:
                raise AssertionError(f"instruction the checker does not know: {ins}")


def run(lines, nb, nk, ntile, ragged=0, turn=0):
    sim = Sim(lines, nb, nk, ntile, ragged)
    sim.turn = turn
    sim.prologue()
    sim.run_tiles()
    return sim


@pytest.fixture(scope="module", params=[(nb, sample) for nb in WIDTHS for sample in (False, True)],
                ids=lambda p: f"{32 * p[0]} tokens, {'sampling' if p[1] else 'greedy'}")
def loop(request):
    nb, sample = request.param
    return nb, listing(nb, sample)[0]


@pytest.mark.parametrize("nk,ntile,ragged", [
    (nk, ntile, 0) for nk in (1, 2, 3, 4, 5, 8, 56, 64) for ntile in (1, 2, 3, 5, 31) if nk < 56 or ntile <= 3] +
    [(5, 1, 7), (5, 2, 1), (5, 4, 255), (6, 3, 128), (9, 2, 77)])
def test_ring_protocol(loop, nk, ntile, ragged):
    nb, lines = loop
    sim = run(lines, nb, nk, ntile, ragged)
    total = nk * ntile
    assert sim.mfma_count == 16 * nb * total and sim.reg["%[g]"] == total    # every step ran both of its groups
    assert sim.started == set(range(32 * nb))                # the last statement started all of its accumulators
    assert sim.next_w_copy == max(total, sim.nw) and sim.next_h_copy == max(total, sim.nh)   # every tile copied exactly once
    assert not sim.unpublished, "copies still unpublished at the end: a later statement would race with them"


def test_the_checker_catches_a_missing_wait(loop):
    """Plant a mistake in a copy of the listing (never in the product): without the vmcnt wait a tile is read
    before it is published, and the checker must say so."""
    nb, lines = loop
    with pytest.raises(AssertionError):
        run([ln for ln in lines if not ln.startswith("s_waitcnt vmcnt")], nb, 5, 3)


def test_the_checker_catches_a_copy_into_a_slot_in_use(loop):
    """Swap the LM-head copy to target the slot being read: the write-after-read rule must fire."""
    nb, lines = loop
    broken = [ln.replace("s_add_u32 %[wdst], %[wdst], 0x8000", "s_add_u32 %[wdst], %[wdst], 0x10000") for ln in lines]
    with pytest.raises(AssertionError, match="may still be reading"):
        run(broken, nb, 4, 3)


def test_the_checker_catches_a_load_right_behind_its_m0_write(loop):
    """What lies between the two moved ahead of both, LM-head and hidden copies alike."""
    nb, lines = loop
    for base in ("%[wdst]", "%[hdst]"):
        with pytest.raises(AssertionError, match="M0"):
            run(without_wait_state(lines, base), nb, 5, 3)


def test_steady_state_spreads_what_lies_between_the_mfmas_evenly(loop):
    """A wave is alone on its SIMD and issues an instruction every few cycles, so more than three instructions
    between two MFMAs (16 cycles apart) delay the second one; a run of 16 no-ops in one gap measured +1.2% on the
    widest tile, the same 16 spread one per gap nothing.  In the steady-state body no gap of a group holds more than its
    share, rounded up (three and four token blocks: two instructions), the sync between the two groups of a step is
    two instructions (wait + barrier), and the only branch taken is the back edge at the end of the body."""
    nb, prog = loop
    start = next(i for i, ln in enumerate(prog) if ln.startswith("Lsteady"))
    end = next(i for i, ln in enumerate(prog) if ln.startswith("Lleave"))
    body = prog[start + 1:end]
    sync = body.index("s_barrier")
    assert body.count("s_barrier") == 1 and body[0] == "s_waitcnt lgkmcnt(0)" and body[sync - 1].startswith("s_waitcnt vmcnt")
    assert body[-1].startswith("s_cbranch_scc1 Lsteady") and sum(ln.startswith(("s_branch", "s_cbranch")) for ln in body) == 1
    for group in (body[1:sync - 1], body[sync + 1:-1]):
        assert sum(ln.startswith("v_mfma") for ln in group) == 8 * nb and group[0].startswith("v_mfma")
        gaps = " ".join("|" if ln.startswith("v_mfma") else "x" for ln in group).split("|")[1:]
        share = -(-(len(group) - 8 * nb) // (8 * nb))
        assert max(gap.count("x") for gap in gaps) <= share and (nb < 3 or share <= 2)
