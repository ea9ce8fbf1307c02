"""Logits that are not finite.  Ids at minus infinity (a vocabulary's unused rows, say) count for nothing, even where they
are all that a lane holds, against a plain fp64 evaluation; a NaN or a plus infinity shows as NaN in the row's
confidence and log-sum-exp, and in no other row.  Both kernels, greedy and sampled."""
import numpy as np
import pytest
import torch

from paper_2601_06562_amd import binding, workloads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
INF = float("inf")
# rows, d, V, flags: the 4-wave kernel in several widths, with a ragged last tile, the general kernel, a pair of launches
SHAPES = [(20, 320, 1024, 0), (300, 320, 1111, 0), (150, 320, 1024, binding.PLAN_GENERAL_KERNEL), (40, 128, 1000, 0)]
# ... and draws whose units share their scores (tests/test_schedule_host.py holds that they do)
SHAPES += [(1100, 320, 8192, 0), (1100, 320, 8132, 0)]


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


@pytest.mark.parametrize("tau", [0.0, 0.7])
@pytest.mark.parametrize("T,d,V,flags", SHAPES)
def test_what_is_not_a_number_shows_in_its_row(T, d, V, flags, tau):
    print(f"not a number: T={T} d={d} V={V} flags={flags} tau={tau}", flush=True)
    hidden, w = inputs(T, d, V)
    tok, conf, lse = outputs(hidden, w, flags, tau)
    rest = np.arange(T) != 7
    bad = hidden.clone()
    bad[7, 3] = float("nan")                                         # every logit of one row
    t, c, s = outputs(bad, w, flags, tau)
    assert np.isnan(c[7]) and np.isnan(s[7]) and t[7] == 2 ** 31 - 1     # no id has entered
    assert all(np.array_equal(a[rest], b[rest]) for a, b in ((t, tok), (c, conf), (s, lse)))
    bad = w.clone()
    bad[V // 2, 3] = float("nan")                                    # one logit of every row
    t, c, s = outputs(hidden, bad, flags, tau)
    assert np.isnan(c).all() and np.isnan(s).all() and (t != V // 2).all()
    assert np.array_equal(t[tok != V // 2], tok[tok != V // 2])
    bad = w.clone()
    bad[V // 2, 0] = INF
    t, c, s = outputs(hidden, bad, flags, tau)
    assert (t == V // 2).all() and np.isnan(c).all() and np.isnan(s).all()
    bad = w.clone()
    bad[:, 0] = -INF                                                 # nothing to choose from
    t, c, s = outputs(hidden, bad, flags, tau)
    assert (t == 2 ** 31 - 1).all() and not (np.isfinite(c) & (c <= 0)).any() and (s < -1e29).all()


@pytest.mark.parametrize("V", [1, 2, 63, 64, 127, 128, 255, 256, 511, 512, 513])
def test_ids_around_the_powers_of_two(V):
    """The id's share of a packed partial is made from V: the last ids of small vocabularies, both decode modes."""
    T, d = 12, 64
    wl = workloads.small_random(T, d, V, p=1.0, seed=V, device=DEV)
    hidden, w = wl.hidden.clone(), wl.w.clone()
    hidden[:, 0] = 1.0
    w[V - 1, 0] = 30.0                                               # the last id wins every row
    lse = torch.logsumexp(hidden.double() @ w.double().t(), 1).cpu().numpy()
    for tau in (0.0, 0.5):
        t, c, s = outputs(hidden, w, 0, tau)
        assert (t == V - 1).all() and np.abs(s - lse).max() <= 2e-5
