"""Logits that are not finite.  Ids at minus infinity (a vocabulary's unused rows, say) count for nothing, even where they
are all that a lane holds; against a plain fp64 evaluation, on both kernels, greedy and sampled."""
import numpy as np
import pytest
import torch

from paper_2601_06562_amd import binding, workloads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
INF = float("inf")
# rows, d, V, flags: the 4-wave kernel in several widths, with a ragged last tile, the general kernel, a pair of launches
SHAPES = [(20, 320, 1024, 0), (300, 320, 1111, 0), (150, 320, 1024, binding.PLAN_GENERAL_KERNEL), (40, 128, 1000, 0)]


def inputs(T, d, V):
    """Hidden rows whose first element is one: a weight row that starts with an infinity has that infinity as its logit."""
    wl = workloads.small_random(T, d, V, p=1.0, seed=T + V, device=DEV)
    hidden, w = wl.hidden.clone(), wl.w.clone()
    hidden[:, 0] = 1.0
    return hidden, w


def outputs(hidden, w, flags, tau):
    T, d = hidden.shape
    V = w.shape[0]
    op = binding.MaskOnlyLogits(T, d, V, device=DEV, sampling=tau > 0)
    op.plan.flags |= flags
    mask = torch.ones(T, dtype=torch.uint8, device=DEV)
    if tau > 0:
        op.sample_step(hidden, w, mask, tau, 5)
    else:
        op.step(hidden, w, mask)
    torch.cuda.synchronize()
    return op.token.cpu().numpy(), op.conf.cpu().numpy(), op.lse.cpu().numpy()


@pytest.mark.parametrize("tau", [0.0, 0.7])
@pytest.mark.parametrize("T,d,V,flags", SHAPES)
def test_ids_at_minus_infinity(T, d, V, flags, tau):
    print(f"minus infinity: T={T} d={d} V={V} flags={flags} tau={tau}", flush=True)
    hidden, w = inputs(T, d, V)
    for gone in (slice(128, 512), slice(0, 256), slice(3, 4), slice(V - 128, V)):
        some = w.clone()
        some[gone, 0] = -INF
        tok, conf, lse = outputs(hidden, some, flags, tau)
        x = (hidden.double() @ some.double().t()).cpu()
        want = torch.logsumexp(x, 1).numpy()
        picked = x.numpy()[np.arange(T), tok]                        # -inf, and so a failure, for an id that is gone
        assert np.abs(lse - want).max() <= 2e-5, gone
        assert np.allclose(conf, np.exp(picked - want), rtol=2e-5, atol=0), gone
        if tau == 0:
            assert (x.max(1).values.numpy() - picked).max() <= 1e-4, gone
