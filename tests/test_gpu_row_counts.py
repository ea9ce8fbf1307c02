"""The division of the work follows the rows found on the device, not the bound the plan was made for: counts around
the row tiles of a loose plan, on both kernels, greedy and sampled.  The results are the same bits as under a tight
plan (the fold makes them independent of the split), and right against a plain fp64 evaluation."""
import numpy as np
import pytest
import torch

from paper_2601_06562_amd import binding, workloads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("d,V,flags", [(320, 2560, 0), (320, 2560, binding.PLAN_GENERAL_KERNEL), (128, 2500, 0),
                                       (320, 2500, 0), (512, 8192, 0),
                                       # a ragged last tile in the 4-wave kernel: one id more than a tile, one id short
                                       # of a tile, one id in the last tile, fewest K-tiles and more
                                       (320, 257, 0), (576, 2303, 0), (320, 2305, 0), (384, 508, 0), (320, 2308, 0)])
def test_results_are_the_same_bits_for_any_bound(d, V, flags):
    T = 3000
    wl = workloads.small_random(T, d, V, p=1.0, seed=d + V, device=DEV)
    for M in (1, 31, 33, 255, 256, 257, 300, 769, 1500, 2999):
        print(f"row counts d={d} V={V} flags={flags} M={M}", flush=True)
        mask = torch.zeros_like(wl.mask)
        mask[torch.arange(M, device=DEV) * (T // M)] = 1
        outs = []
        for bound, budget in ((T, 0), (M, 0), (T, 140000)):
            for tau in (0.0, 0.7):
                op = binding.MaskOnlyLogits(T, d, V, max_rows=bound, budget_bytes=budget, device=DEV, sampling=tau > 0)
                op.plan.flags |= flags
                if tau > 0:
                    op.sample_step(wl.hidden, wl.w, mask, tau, 99)
                else:
                    op.step(wl.hidden, wl.w, mask)
                torch.cuda.synchronize()
                assert int(op.count.item()) == M
                outs.append(tuple(t[:M].cpu().numpy() for t in (op.token, op.conf, op.lse)))
        for k in (2, 3, 4, 5):
            for a, b in zip(outs[k % 2], outs[k]):
                assert np.array_equal(a, b), (M, k)
        if d < 320 or V % 4 == 0:                                     # (else another kernel serves the ragged tile)
            assert np.array_equal(outs[0][2], outs[1][2])            # the log-sum-exp does not depend on the draw
        rows = torch.nonzero(mask).flatten()
        x = wl.hidden[rows].double() @ wl.w.double().t()
        lse = torch.logsumexp(x, 1).cpu().numpy()
        assert np.abs(outs[0][2] - lse).max() <= 2e-5
        picked = x.gather(1, torch.as_tensor(outs[0][0], device=DEV).long()[:, None])[:, 0]
        assert float((x.max(1).values - picked).max()) <= 1e-4
