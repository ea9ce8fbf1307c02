"""The part of the sampling statements that takes over the published scores, of every width, on the CPU: the lanes of a column
end with the larger of their own best and a float just below what is published for the column's row, whatever its sign; rows
that pad a tile read the last row's word, and nothing outside the wave's rows is read."""
import os

import numpy as np
import pytest

from test_w4_loop_protocol import GEN, gen, listing
from test_w4_tile_reduce import Wave

NEG = -2.0 ** 100


def score_order(x):
    """The kernel's word for a score: integers in the scores' order."""
    b = np.asarray(x, np.float32).view(np.int32)
    return b ^ ((b >> 31) & 0x7FFFFFFF)


class Taking(Wave):
    def __init__(self, n, published):
        super().__init__(n, np.zeros((256, n), np.float32))
        self.published = published

    def step(self, ins):
        op, _, rest = ins.partition(" ")
        a = [x.strip() for x in rest.split(",")]
        if op == "v_min_i32":
            self.iset(a[0], np.minimum(self.iget(a[1]).view(np.int32), self.iget(a[2]).view(np.int32)).view(np.uint32))
        elif op == "v_ashrrev_i32":
            self.iset(a[0], (self.iget(a[2]).view(np.int32) >> int(a[1])).view(np.uint32))
        elif op == "global_load_dword":
            assert a[2] == "%[rb] sc0"
            at = self.iget(a[1])
            assert np.all(at % 4 == 0) and np.all(at // 4 < len(self.published))
            self.reg[a[0]] = score_order(self.published[at // 4]).view(np.uint32).copy()
            self.pending_lds.add(a[0])
        elif op == "s_waitcnt" and rest == "vmcnt(0)":
            self.pending_lds.clear()
        elif op == "ds_bpermute_b32" and "offset:" in rest:
            data, _, offset = a[2].partition(" offset:")
            self.iset(a[0], self.iget(data)[((self.iget(a[1]) + int(offset)) >> 2) % self.n])
            self.pending_lds.add(a[0])
        else:
            super().step(ins)


@pytest.mark.parametrize("rows", [1, 5, 16, 17, 63, 64, 65, 100, 127, 128])
@pytest.mark.parametrize("nb", range(1, 9))
def test_published_scores_are_taken_over(nb, rows):
    rows = min(rows, 16 * nb)
    rng = np.random.default_rng(nb * 1000 + rows)
    published = rng.standard_normal(rows).astype(np.float32) * 20
    published[::3] = np.float32(NEG)                             # nothing published
    published[1::7] = np.float32(np.inf)
    published[2::11] = 0.0
    published[5::13] = -0.0
    published[7::17] = np.float32(1e-45)
    own = (rng.standard_normal((nb, 64)) * 20).astype(np.float32)
    own[0] = NEG
    _, ragged, red = listing(nb, True)
    at = next(i for i, ln in enumerate(ragged) if ln.startswith("Ltake"))
    assert ragged[at - 1].startswith("s_branch Lwhole") and ragged[-1].startswith("Lwhole")
    w = Taking(64, published)
    w.iset("%[first]", np.full(64, gen.TAKE))
    w.iset("%[rl]", np.full(64, rows - 1))
    for tb in range(nb):
        w.fset(f"%[ym{tb}]", own[tb])
    w.run(ragged)
    for tb in range(nb):
        row = np.minimum(16 * tb + np.arange(64) % 16, rows - 1)
        best = published[row]
        got = w.fget(f"%[ym{tb}]")
        taken = got != own[tb]
        assert np.all(got[taken] > own[tb][taken]) and np.all(got[taken] < best[taken]), tb   # the very same score still wins
        below = best
        for _ in range(3):
            below = np.nextafter(below, np.float32(-np.inf))
        assert np.all(got >= np.where(best == NEG, own[tb], np.maximum(own[tb], below))), tb


def test_words_are_in_the_scores_order():
    x = np.array([-np.inf, -3e38, NEG, -300.5, -1.0, -1e-45, -0.0, 0.0, 1e-45, 1.0, 300.5, 3e38, np.inf], np.float32)
    k = score_order(x)
    assert np.all(k[1:] > k[:-1])
    kernel = open(os.path.join(os.path.dirname(GEN), "mosaic_logits.hip")).read()
    assert "return b ^ (int)((uint32_t)(b >> 31) >> 1);" in kernel             # the same function of the bits
