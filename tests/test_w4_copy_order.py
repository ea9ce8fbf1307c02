"""The K-loops with a unit's LM-head copies in an order of its own (copy i brings piece i ^ turn to its place in LDS), on the
CPU: both loops are interpreted as in test_w4_loop_protocol.py and test_w4_pair_order.py, with %[wdst] as the kernel hands it
in for that order and %[woff i] standing for piece i ^ turn, and every piece has to come to lie in its own KiB, once.  The
kernel's side of it, the offsets and the prologue's copies, is held to the same functions of the order."""
import os
import re

import pytest

import test_w4_loop_protocol as protocol
import test_w4_pair_order as pair_order

TURNS = (2, 4, 6)
SHAPES = [(1, 1, 0), (2, 3, 0), (5, 4, 0), (5, 2, 1), (9, 2, 77)]
NARROWER = range(1, 8)


def interpret(lines, nb, *shape, **kw):
    return (pair_order if nb in pair_order.WIDTHS else protocol).run(lines, nb, *shape, **kw)


@pytest.mark.parametrize("turn", TURNS)
@pytest.mark.parametrize("nb", NARROWER)
def test_turned_copies_come_to_lie_in_their_places(nb, turn):
    for sample in (False, True):
        lines = protocol.listing(nb, sample)[0]
        for shape in SHAPES:
            interpret(lines, nb, *shape, turn=turn)


@pytest.mark.parametrize("nb", NARROWER)
def test_places_by_addition_are_caught(nb):
    """Planted: the place of copy i as %[wdst] + 1024 i, which leaves the wave's 8 KiB."""
    lines = [ln.replace("s_xor_b32 m0,", "s_add_u32 m0,") for ln in protocol.listing(nb)[0]]
    interpret(lines, nb, 5, 3)                                  # in the plain order it is the same
    with pytest.raises(AssertionError, match="not to its own KiB"):
        interpret(lines, nb, 5, 3, turn=6)


@pytest.mark.parametrize("nb", NARROWER)
def test_offsets_in_another_order_than_the_places_are_caught(nb, monkeypatch):
    """Planted in the checker's glue: offsets in the plain order under places in the unit's."""
    monkeypatch.setattr(protocol.Sim, "source_piece", lambda self, operand, offset: int(re.search(r"\d", offset).group()))
    with pytest.raises(AssertionError, match="not to its own KiB"):
        interpret(protocol.listing(nb)[0], nb, 5, 3, turn=2)


def test_the_kernels_orders():
    """The kernel's expressions, evaluated: turns are even, so that a piece keeps the swizzle of its parity, within a wave's
    eight pieces, and the place that the loop makes of %[wdst] is the one the prologue copies the piece to."""
    kernel = open(os.path.join(os.path.dirname(protocol.GEN), "mosaic_logits.hip")).read()
    for expression in ("const int turn = NB < 8 ? (tt & 1) * 4 + (tt & 2) : 0;",
                       "woff[i] = wlane[i & 1] + (uint32_t)(8 * (i ^ turn)) * w_row_bytes;",
                       "(lds_ptr_t)(dst + (i ^ turn) * 1024)",
                       "st_wdst = (uint32_t)((gw % NW) * kLmHeadSlot) + w_dst + (uint32_t)turn * 1024u;"):
        assert kernel.count(expression) == 1, expression
    for tt in range(8):
        turn = (tt & 1) * 4 + (tt & 2)
        assert turn in (0, *TURNS) and sorted(i ^ turn for i in range(8)) == list(range(8))
        for slot in range(4):
            for wave in range(4):
                base = slot * 0x8000 + wave * 0x2000
                for i in range(8):
                    assert (base + 1024 * turn) ^ (1024 * i) == base + 1024 * (i ^ turn) and (i ^ turn) % 2 == i % 2
