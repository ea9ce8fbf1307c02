"""The division of the work follows the rows found on the device, not the bound the plan was made for: counts around
the row tiles of a loose plan, on both kernels, greedy and sampled.  The results are the same bits as under a tight
plan (the fold makes them independent of the split), and right against a plain fp64 evaluation.  Hidden tensors of
4 GiB or more with a ragged vocabulary: up to three launches share one division there."""
import numpy as np
import pytest
import torch

from paper_2601_06562_amd import binding, workloads
from test_gpu_full_size import span_flag

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


@pytest.mark.parametrize("V", [2560, 2500])
def test_a_plans_grid_may_exceed_its_units(V):
    T, d = 700, 128
    wl = workloads.small_random(T, d, V, p=0.7, seed=V, device=DEV)
    outs = []
    for grid in (0, 1 << 20, 1 << 30):
        print(f"grid {grid} V={V}", flush=True)
        op = binding.MaskOnlyLogits(T, d, V, device=DEV)
        op.plan.grid = grid or op.plan.grid
        op.step(wl.hidden, wl.w, wl.mask)
        torch.cuda.synchronize()
        outs.append([t[:int(op.count.item())].cpu().numpy() for t in (op.token, op.conf, op.lse)])
    assert all(np.array_equal(a, b) for out in outs[1:] for a, b in zip(outs[0], out))


@pytest.mark.parametrize("V", [50257, 4096])
def test_a_pair_of_launches_beyond_4_gib_shares_one_division(V):
    """A ragged vocabulary served by a pair of launches (fewer than five K-tiles; under sampling also V % 4 != 0), in a
    hidden tensor beyond 4 GiB: where the list has a 4 GiB gap inside the rows of one wave the general kernel takes the
    4-wave kernel's place, in 49 vocabulary splits for these 769 rows instead of 40, and the launch for the ragged tile
    has to store behind those.  And a vocabulary without one, whose width and division are searched for the rows found
    all the same.  Expected: the general kernel on the same rows gathered into a small tensor."""
    T, d = (1 << 23) + 8192, 256
    gen = torch.Generator(device=DEV)
    gen.manual_seed(workloads.BASE_SEED + 79)
    hidden = torch.empty((T, d), dtype=torch.bfloat16, device=DEV)
    for r in range(0, T, 1 << 20):
        hidden[r:r + (1 << 20)].normal_(generator=gen)
    w = workloads._normal_bf16(V, d, d ** -0.5, gen, torch.device(DEV))
    assert T * d * 2 > 1 << 32
    for M, bound in ((769, 769), (513, 4096), (40, 40), (40, 5000)):
        lists = {1: torch.cat([torch.arange(3, 20), torch.arange(T - (M - 17) * 3, T, 3)]),   # the gap in the first group
                 0: torch.arange(T - M * 3, T, 3)}
        for flag, pos in lists.items():
            pos = pos.to(DEV)
            mask = torch.zeros(T, dtype=torch.uint8, device=DEV)
            mask[pos] = 1
            rows = hidden[pos].contiguous()
            small = torch.arange(M, dtype=torch.int32, device=DEV)
            lse = torch.logsumexp(rows.double() @ w.double().t(), 1).cpu().numpy()
            for tau in (0.0, 0.8):
                print(f"pair beyond 4 GiB: M={M} bound={bound} flag={flag} tau={tau}", flush=True)
                op = binding.MaskOnlyLogits(T, d, V, max_rows=bound, device=DEV, sampling=tau > 0)
                name = binding.mosaic_masked_logits_kernel_name(1000, d, d, V, op.plan, tau > 0)
                assert ("ragged last vocabulary tile" in name) == (V % 256 != 0)
                ref = binding.MaskOnlyLogits(M, d, V, device=DEV, sampling=tau > 0)
                ref.plan.flags |= binding.PLAN_GENERAL_KERNEL
                if tau > 0:
                    op.sample_step(hidden, w, mask, tau, 99)
                    binding.mosaic_masked_logits_sample(rows, w, small, op.count, M, tau, 99, ref.token, ref.conf,
                                                        ref.lse, ref.plan, ref.workspace, noise_idx=op.idx)
                else:
                    op.step(hidden, w, mask)
                    binding.mosaic_masked_logits_reduce(rows, w, small, op.count, M, ref.token, ref.conf, ref.lse,
                                                        ref.plan, ref.workspace)
                torch.cuda.synchronize()
                assert int(op.count.item()) == M and span_flag(op) == flag
                what = (M, bound, flag, tau)
                assert torch.equal(op.token[:M], ref.token[:M]), what
                assert torch.allclose(op.conf[:M], ref.conf[:M], rtol=1e-5, atol=0), what    # sums in another order
                assert np.abs(op.lse[:M].cpu().numpy() - lse).max() <= 2e-5, what
    del hidden
    torch.cuda.empty_cache()
