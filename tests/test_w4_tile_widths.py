"""The generated statements of every width of the row tile (32 to 256 tokens), on the CPU: the reduction of each
against the definition of the triples it yields, the ragged last tile's included, and, instruction by instruction,
against the widest tile's on this width's accumulators.  The sampling reduction with a quad's own bound draws what it
draws without, and leaves few quads to the exact path.  (The K-loops: test_w4_loop_protocol.py, test_w4_pair_order.py.)"""
import re

import numpy as np
import pytest

from test_w4_loop_protocol import gen, listing, writes_m0


@pytest.mark.parametrize("nb", range(1, 9))
def test_copies_keep_the_wait_state_behind_their_m0_write(nb):
    """A direct-to-LDS load needs an instruction between the write of M0 and itself."""
    for sample in (False, True):
        loop, _, _ = listing(nb, sample)
        writes = [ln for ln in loop if writes_m0(ln)]
        loads = sum(ln.startswith("global_load_lds") for ln in loop)
        assert len(writes) == loads and len({ln.split()[0] for ln in writes}) == 2   # LM-head and hidden copies: none is overlooked
        for a, b in zip(loop, loop[1:]):
            assert not (writes_m0(a) and b.startswith("global_load_lds"))


@pytest.mark.parametrize("sample", [False, True])
@pytest.mark.parametrize("nb", range(1, 8))
def test_reduction_of_every_width_is_the_widest_tiles(nb, sample):
    plain = lambda ln: re.sub(r"\bL([a-z]+)\d+_%=", r"L\1", ln)
    _, _, wide = listing(8, sample)
    _, _, red = listing(nb, sample)

    def widen(m):                       # accumulator (bi*nb + tb)*4 + r of this width -> (bi*8 + tb)*4 + r
        block, r = divmod(int(m.group(1)), 4)
        return f", a{(block // nb * 8 + block % nb) * 4 + r}"
    got = [plain(re.sub(r", a(\d+)$", widen, ln)) if ln.startswith("v_accvgpr_read") else plain(ln) for ln in red]
    wide = [plain(ln) for ln in wide]

    def columns(prog):                  # cut at the first accumulator read of each column; drop what follows the last
        starts = [i for i, ln in enumerate(prog) if re.match(r"v_accvgpr_read_b32 v112,", ln)]
        head = starts[0]
        while sample and not prog[head].startswith("ds_bpermute_b32 v177"):
            head -= 1
        back = starts[0] - head
        return prog[:head], [prog[a - back:b - back] for a, b in zip(starts, starts[1:])], prog[starts[-1] - back:]
    (head, cols, last), (whead, wcols, _) = columns(got), columns(wide)
    assert head == whead and cols == wcols[:nb - 1]
    body = wcols[nb - 1]
    assert last[:len(body)] == body
    rest = last[len(body):]
    if not sample:
        assert rest == []
    else:                               # the exact paths out of line: one block per quad, the widest tile's first ones
        at = next(i for i, ln in enumerate(wide) if ln == "s_branch Ldone")
        names = lambda ln: re.sub(r"L(slow|flush|back|queue|full|nothing)\b", r"L", ln)
        assert rest[0] == "s_branch Ldone" and rest[-1] == "Ldone:"
        assert [names(x) for x in rest[1:-1]] == [names(x) for x in wide[at + 1:at + len(rest) - 1]]


@pytest.mark.parametrize("tau", [1.0, 0.3])
def test_a_quads_own_bound_changes_no_draw(tau):
    import test_w4_tile_reduce as reduce
    reduce.TEMPS.update(gen.SAMPLE_TEMPS)
    rng = np.random.default_rng(int(10 * tau))
    n, seed = 64, 0x0F1E2D3C4B5A6978
    lane = np.arange(n, dtype=np.uint32)
    vb = np.full(n, 11 * 256, np.uint32) + 4 * (lane >> 4)
    pos = [rng.integers(0, 4096, 16).astype(np.uint32)[lane % 16] for _ in range(8)]
    i0 = (300000 + rng.permutation(8 * n).reshape(8, n)).astype(np.uint32)
    xa0 = rng.standard_normal((8, n)).astype(np.float32)
    tight = [ln for part in listing(8, True)[1:] for ln in part]
    gen.SHAPE["tight"] = False
    plain = [ln for part in listing(8, True)[1:] for ln in part]
    gen.SHAPE["tight"] = True
    for best in (-2.0 ** 100, 2 + 2 * tau, 3 + 5 * tau, 3 + 9 * tau):   # fresh columns, then ever later in a split
        for planted in (False, True):
            agpr = reduce.planted_tile(rng, n) if planted else rng.standard_normal((256, n)).astype(np.float32)
            ym0 = np.full((8, n), best, np.float32)
            ym0[:, lane % 16 == 5] = -2.0 ** 100                        # one token is fresh in any case
            out = {}
            for key, red, exact in (("exact", plain, True), ("plain", plain, False), ("tight", tight, False)):
                out[key] = reduce.sampling_wave(red, agpr, ym0, xa0, i0, pos, vb, seed, tau, force_exact=exact)
            for tb in range(8):
                assert reduce.token_level(out["tight"], tb) == reduce.token_level(out["exact"], tb), (best, planted, tb)
                for name in ("m", "s"):
                    assert np.array_equal(out["tight"].reg[f"%[{name}{tb}]"], out["exact"].reg[f"%[{name}{tb}]"])
            assert out["tight"].flushes <= out["plain"].flushes and out["tight"].fulls <= out["plain"].fulls
            print(tau, best, planted, *((k, o.issued, o.slow_taken, o.flushes, o.fulls) for k, o in out.items()))


def reduce_wave(nb, sample, agpr, vb, first, tau=0.8):
    """One wave's reduction, on nothing drawn before: (m, s, i) of every column, or (m, s, ym, xa, i)."""
    import test_w4_tile_reduce as reduce
    reduce.TEMPS.update(gen.SAMPLE_TEMPS)
    n = agpr.shape[1]
    w = reduce.Wave(n, agpr.copy())
    for name, v in (("vb", vb), ("first", np.full(n, first)), ("seed_lo", np.full(n, 77)), ("seed_hi", np.full(n, 5)),
                    ("pm0", np.full(n, 0xD2511F53)), ("pm1", np.full(n, 0xCD9E8D57))):
        w.iset(f"%[{name}]", v)
    w.fset("%[itl]", np.full(n, np.float32(1.4426950408889634) / np.float32(tau)))
    w.fset("%[tau]", np.full(n, tau))
    for tb in range(nb):
        if sample:
            w.fset(f"%[ym{tb}]", np.full(n, -2.0 ** 100)), w.fset(f"%[xa{tb}]", np.zeros(n))
            w.iset(f"%[i{tb}]", np.full(n, 0x7FFFFFFF))
            w.iset(f"%[pos{tb}]", 1000 * tb + np.arange(n) % 16)
    _, ragged, red = listing(nb, sample)
    w.run(ragged + red)
    return [[w.reg[f"%[{name}{tb}]"].view(np.uint32 if name == "i" else np.float32)
             for name in (("m", "s", "ym", "xa", "i") if sample else ("m", "s", "i"))] for tb in range(nb)]


def check_triples(nb, sample, got, agpr, taken_out):
    """Every column's triple against its definition in 64 bits; taken_out: bool[32, n], elements that do not count."""
    for tb in range(nb):
        x = np.stack([agpr[(el // 4 * nb + tb) * 4 + el % 4] for el in range(32)]).astype(np.float64)
        x[taken_out] = -2.0 ** 100
        t = np.maximum(x.max(axis=0), -2.0 ** 100)
        with np.errstate(over="ignore"):
            want = np.exp(x - t).sum(axis=0)
        assert np.array_equal(got[tb][0], t.astype(np.float32)), tb
        assert np.all(np.abs(got[tb][1] - want) <= 2e-6 * want), (tb, got[tb][1], want)
        if not sample:
            sel = (x == t).argmax(axis=0)
            some = t > -2.0 ** 100                            # (else the kernel takes no id from it)
            code = 16 * (sel // 4) + sel % 4
            assert np.array_equal((got[tb][2] & 0xFF)[some], code[some]), tb


@pytest.mark.parametrize("sample", [False, True])
@pytest.mark.parametrize("nb", range(1, 9))
def test_ids_at_minus_infinity_count_for_nothing(nb, sample):
    """A lane whose ids are all at minus infinity (a vocabulary's unused rows, say) yields an empty triple: with its
    own maximum taken from its exponents its sum is NaN."""
    rng = np.random.default_rng(nb)
    n = 64
    agpr = rng.standard_normal((256, n)).astype(np.float32)
    agpr[:, 7] = -np.inf
    agpr[:17 * nb, 9] = -np.inf
    agpr[5, 11] = -np.inf
    got = reduce_wave(nb, sample, agpr, np.zeros(n), 0)
    check_triples(nb, sample, got, agpr, np.zeros((32, n), bool))
    for tb in range(nb):
        assert got[tb][1][7] == 0
        if sample:
            assert got[tb][4][7] == 0x7FFFFFFF and got[tb][2][7] == -2.0 ** 100


@pytest.mark.parametrize("sample", [False, True])
@pytest.mark.parametrize("nb", range(1, 9))
def test_a_tiles_triple_and_the_ids_counted_before(nb, sample):
    """The reduction of every width against its definition: a whole tile, and the ragged last one, which lies over the
    vocabulary's last 256 ids and of which `left` have not been counted (1: one; 256: a whole tile, %[first] is 0).  Ties
    go to the lowest id.  The interpreter checks the distances between comparisons and their use on the way."""
    rng = np.random.default_rng(17 * nb)
    n = 64
    lane = np.arange(n)
    for left in (256, 255, 200, 128, 44, 4, 1):
        for half in (0, 128):                                 # the two waves' ids
            vb = 1000 * 256 + left - 256 + half + 4 * (lane >> 4)
            first = 0 if left == 256 else 1000 * 256
            agpr = rng.standard_normal((256, n)).astype(np.float32) * 3
            for k in range(3):                                # exact ties
                agpr[rng.integers(0, 32 * nb, n), lane] = 20
            code = np.array([16 * (el // 4) + el % 4 for el in range(32)])[:, None]
            taken_out = vb + code < first
            got = reduce_wave(nb, sample, agpr, vb, first)
            if not sample:
                for col in got:
                    col[2] -= vb.astype(np.uint32)
            check_triples(nb, sample, got, agpr, taken_out)
            for m, s, ym, xa, i in got if sample else ():
                some = ~taken_out.all(axis=0)
                assert np.all(i[some] != 0x7FFFFFFF) and np.all((i >= first)[some]) and np.all(i[~some] == 0x7FFFFFFF)
                assert np.all(np.abs(xa[some]) < 100) and np.all(xa[some] <= m[some])
