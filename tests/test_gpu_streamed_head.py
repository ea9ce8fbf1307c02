"""One row tile against an LM head beyond the memory-side cache: its copies carry the nt bit there, in code of their own
for every width.  Expected: the same bits as where the same rows share the LM head with more rows than one tile holds
(plain copies), greedy and drawn, whole and ragged vocabulary; and a plain evaluation for some of the rows.  That the
listed steps are lone row tiles, of every width, is held by tests/test_schedule_host.py; but for the drawn steps of more than
224 rows at d = 1024, which take two (plain copies again): at d = 2048 these, too, are lone ones."""
import pytest
import torch

from paper_2601_06562_amd import binding, workloads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
STREAM_BYTES = 288 << 20
T = 600                                                            # three row tiles of 256 rows
ROWS = (1, 31, 32, 33, 64, 65, 96, 128, 129, 160, 192, 193, 224, 225, 256)
# (d, V): the smallest heads that stream at d = 1024, whole and with a ragged tile; the same at d = 2048 and 512 tiles.
# Rows of the greedy and of the drawn steps.
STEPS = {(1024, 147456 + 256): (ROWS, ROWS), (1024, 147456 + 8): (ROWS, ROWS),
         (2048, 131072): ((), (225, 255, 256)), (2048, 131064): ((), (225, 255, 256))}


@pytest.mark.parametrize("d,V", STEPS)
def test_a_streamed_head_gives_the_same_bits(d, V):
    assert STREAM_BYTES < 2 * V * d and (d > 1024 or 2 * V * d < STREAM_BYTES + (1 << 20))
    wl = workloads.small_random(T, d, V, p=1.0, seed=V, device=DEV)

    def run(rows, tau):
        print(f"streamed head V={V} rows={rows} tau={tau}", flush=True)
        mask = torch.zeros_like(wl.mask)
        mask[:rows] = 1
        op = binding.MaskOnlyLogits(T, d, V, max_rows=rows, device=DEV, sampling=tau > 0)
        op.sample_step(wl.hidden, wl.w, mask, tau, 5) if tau > 0 else op.step(wl.hidden, wl.w, mask)
        torch.cuda.synchronize()
        assert int(op.count.item()) == rows
        return [t[:rows].clone() for t in (op.token, op.conf, op.lse)]

    for tau, counts in zip((0.0, 0.8), STEPS[d, V]):
        want = run(T, tau)                                     # several row tiles
        for rows in counts:
            assert all(torch.equal(a, b[:rows]) for a, b in zip(run(rows, tau), want)), (rows, tau)
        x = wl.hidden[:40].double() @ wl.w.double().t()
        assert float((want[2][:40] - torch.logsumexp(x, 1)).abs().max()) <= 2e-5
        if tau == 0:
            picked = x.gather(1, want[0][:40].long()[:, None])[:, 0]
            assert float((x.max(1).values - picked).max()) <= 1e-4
