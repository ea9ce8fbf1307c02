"""A draw in which the units of a row share the best scores they have reached, against the same rows drawn a few at a time, in
units of 32 rows and one or two vocabulary tiles, which share nothing: the same bits.  The array that the scores are shared in,
the confidences', holds large values ahead of every draw: taken for scores they would leave nothing to be drawn."""
import pytest
import torch

from paper_2601_06562_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def drawn(op, hidden, w, gather, pos, tau, seed):
    n = gather.numel()
    op.count.fill_(n)
    op.conf.fill_(1e30)
    binding.mosaic_masked_logits_sample(hidden, w, gather, op.count, op.max_rows, tau, seed, op.token, op.conf, op.lse,
                                        op.plan, op.workspace, noise_idx=pos)
    return [x[:n].clone() for x in (op.token, op.conf, op.lse)]


# rows: one row tile short of full and past it, several rounds of units (9000), a bound far above the rows; logits all below
# zero (whose scores are not shared), flat ones, ones with a certain id
@pytest.mark.parametrize("rows, V, tau, offset", [(1537, 8192, 1.0, 0.0), (2600, 8192, 0.7, 0.0), (2600, 8192, 0.7, -300.0),
                                                  (9000, 8192, 0.5, 0.0), (2111, 8188, 1.0, 0.0), (2111, 8130, 0.9, 0.0)])
def test_shared_bounds_change_no_draw(rows, V, tau, offset):
    d, T = 512, rows + 100
    gen = torch.Generator(device=DEV)
    gen.manual_seed(rows + V)
    w = (torch.randn((V, d), generator=gen, device=DEV) * d ** -0.5).to(torch.bfloat16)
    hidden = torch.randn((T, d), generator=gen, device=DEV)
    certain = torch.rand((T, 1), generator=gen, device=DEV) * 20
    hidden += certain * w[torch.randint(0, V, (T,), generator=gen, device=DEV)]
    if offset:
        w[:, 0], hidden[:, 0] = 1.0, offset
    hidden = hidden.to(torch.bfloat16)
    gather = torch.randperm(T, generator=gen, device=DEV)[:rows].to(torch.int32).sort().values
    pos = gather + 7
    want = []
    few = binding.MaskOnlyLogits(T, d, V, max_rows=32, device=DEV, sampling=True)
    assert (V + 255) // 256 <= 2 * few.plan.vocab_splits          # units of two tiles at most
    for r in range(0, rows, 32):
        want.append(drawn(few, hidden, w, gather[r:r + 32], pos[r:r + 32], tau, 41))
    want = [torch.cat(x) for x in zip(*want)]
    for bound in (rows, T):
        op = binding.MaskOnlyLogits(T, d, V, max_rows=bound, device=DEV, sampling=True)
        got = drawn(op, hidden, w, gather, pos, tau, 41)
        torch.cuda.synchronize()
        assert torch.equal(got[0], want[0])
        assert (got[2] != want[2]).sum() <= 1 and torch.allclose(got[2], want[2], rtol=2e-7, atol=0)   # a last bit, once in a million
        assert torch.allclose(got[1], want[1], rtol=1e-6, atol=0)


@pytest.mark.parametrize("rows", [97, 180, 256])
def test_units_of_two_tiles_share_too(rows):
    test_shared_bounds_change_no_draw(rows, 130816, 0.7, 0.0)      # 511 vocabulary tiles, one row tile
