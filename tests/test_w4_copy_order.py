"""The K-loops with a unit's LM-head copies in an order of its own (copy i brings piece i ^ turn to its place in LDS), on the
CPU: both loops are interpreted as in test_w4_loop_protocol.py and test_w4_pair_order.py, with the ring's place handed in as the
kernel does for that order, and every piece has to come to lie where the order says."""
import pytest

import test_w4_loop_protocol as protocol
import test_w4_pair_order as pair_order

TURNS = (2, 4, 6)
SHAPES = [(1, 1, 0), (2, 3, 0), (5, 4, 0), (5, 2, 1), (9, 2, 77)]


@pytest.mark.parametrize("turn", TURNS)
@pytest.mark.parametrize("nb", [n for n in pair_order.WIDTHS if n < 8])
def test_pair_order_with_turned_copies(nb, turn, monkeypatch):
    seen = set()

    class Turned(pair_order.PairWave):
        def prologue(self):
            super().prologue()
            self.reg["%[wdst]"] += 1024 * turn

        def copy(self, op):
            if op == "W":
                place = self.reg["m0"]
                seen.add(place % 0x2000 // 1024)
                self.reg["m0"] = place ^ 1024 * turn          # where it would go in the plain order
                super().copy(op)
                self.reg["m0"] = place
            else:
                super().copy(op)
    monkeypatch.setattr(pair_order, "PairWave", Turned)
    for shape in SHAPES:
        pair_order.run(pair_order.listing(nb), nb, *shape)
    assert seen == set(range(8))                              # within the wave's 8 KiB


@pytest.mark.parametrize("turn", TURNS)
@pytest.mark.parametrize("nb", protocol.WIDTHS)
def test_the_loops_of_the_narrow_widths_with_turned_copies(nb, turn):
    ins = [ln for ln in protocol.listing(nb)[0] if "m0" in ln and "%[wdst]" in ln]
    pieces = [int(ln.split(",")[-1]) // 1024 for ln in ins]
    assert ins and all(ln.startswith("s_xor_b32 m0, %[wdst], ") for ln in ins) and len(pieces) % 8 == 0
    for k in range(0, len(pieces), 8):
        assert pieces[k:k + 8] == list(range(8))              # place = wdst ^ 1024 i, so turned by wdst's low bits alone
        assert sorted((1024 * turn ^ 1024 * i) // 1024 for i in pieces[k:k + 8]) == list(range(8))
