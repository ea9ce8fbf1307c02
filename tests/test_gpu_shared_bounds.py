"""A draw in which the units of a row share the best scores they have reached, against the same rows drawn a few at a time, in
units of 32 rows and one or two vocabulary tiles, which share nothing: the same ids, and the same bits but for a last one.  The
array that the scores are shared in, the confidences', holds large values ahead of every draw: taken for scores they would leave
nothing to be drawn.  That the listed draws share and the ones they are held against do not is held by
tests/test_schedule_host.py."""
import pytest
import torch

from paper_2601_06562_amd import binding
from test_gpu_full_size import span_flag

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
D = 512
FEW = 32
# rows, V, temperature, offset of all logits: one row tile short of full and past it, two rounds of units (17000: 67 row tiles in
# four splits), ragged vocabularies, the last one served by a pair of launches; logits all below zero, flat ones and ones with
# a certain id
CASES = [(1537, 8192, 1.0, 0.0), (2600, 8192, 0.7, 0.0), (2600, 8192, 0.7, -300.0), (9000, 8192, 0.5, 0.0),
         (17000, 8192, 0.7, 0.0), (2111, 8188, 1.0, 0.0), (2111, 8130, 0.9, 0.0)]
TWO_TILES, TWO_TILES_V = (40, 64, 97, 180, 256), 130816             # 511 vocabulary tiles, one row tile
CHUNKED = (2600, 8192, 20000)                                       # rows, V, budget
GRAPH = (2600, 8192)
BEYOND_4_GIB = ((1 << 22) + 4096, 8192, 2200)                       # T, V, rows
SHARING = [(D, V, bound, rows, 0) for rows, V, _, _ in CASES for bound in (rows, rows + 100)]
SHARING += [(D, TWO_TILES_V, bound, rows, 0) for rows in TWO_TILES for bound in (rows, rows + 100)]
SHARING += [(D, CHUNKED[1], CHUNKED[0], CHUNKED[0], CHUNKED[2]), (D, GRAPH[1], GRAPH[0], GRAPH[0], 0),
            (D, BEYOND_4_GIB[1], BEYOND_4_GIB[2], BEYOND_4_GIB[2], 0)]
SHARING += [(320, V, 1100, 1100, 0) for V in (8192, 8132)]          # tests/test_gpu_non_finite.py
ALONE = [(D, V, FEW, rows, 0) for V in sorted({c[1] for c in CASES}) + [TWO_TILES_V] for rows in (1, 8, FEW)]


def inputs(T, V, offset=0.0):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(T + V)
    w = (torch.randn((V, D), generator=gen, device=DEV) * D ** -0.5).to(torch.bfloat16)
    hidden = torch.randn((T, D), generator=gen, device=DEV)
    certain = torch.rand((T, 1), generator=gen, device=DEV) * 20
    hidden += certain * w[torch.randint(0, V, (T,), generator=gen, device=DEV)]
    if offset:
        w[:, 0], hidden[:, 0] = 1.0, offset
    return hidden.to(torch.bfloat16), w, gen


def drawn(op, hidden, w, gather, pos, tau, seed):
    n = gather.numel()
    op.count.fill_(n)
    op.conf.fill_(1e30)
    binding.mosaic_masked_logits_sample(hidden, w, gather, op.count, op.max_rows, tau, seed, op.token, op.conf, op.lse,
                                        op.plan, op.workspace, noise_idx=pos)
    return [x[:n].clone() for x in (op.token, op.conf, op.lse)]


def drawn_alone(hidden, w, gather, pos, tau, seed):
    few = binding.MaskOnlyLogits(hidden.shape[0], D, w.shape[0], max_rows=FEW, device=DEV, sampling=True)
    out = [drawn(few, hidden, w, gather[r:r + FEW], pos[r:r + FEW], tau, seed) for r in range(0, gather.numel(), FEW)]
    return [torch.cat(x) for x in zip(*out)]


def check_same(got, want):
    assert torch.equal(got[0], want[0])
    for a, b in zip(got[1:], want[1:]):                             # another split: a last bit, once in a million rows
        assert (a != b).sum() <= 1 and torch.allclose(a, b, rtol=2.5e-7, atol=0)


@pytest.mark.parametrize("rows, V, tau, offset", CASES)
def test_shared_bounds_change_no_draw(rows, V, tau, offset):
    print(f"shared bounds: rows={rows} V={V} tau={tau} offset={offset}", flush=True)
    T = rows + 100
    hidden, w, gen = inputs(T, V, offset)
    gather = torch.randperm(T, generator=gen, device=DEV)[:rows].to(torch.int32).sort().values
    pos = gather + 7
    want = drawn_alone(hidden, w, gather, pos, tau, 41)
    for bound in (rows, T):
        op = binding.MaskOnlyLogits(T, D, V, max_rows=bound, device=DEV, sampling=True)
        for _ in range(2):
            got = drawn(op, hidden, w, gather, pos, tau, 41)
            torch.cuda.synchronize()
            check_same(got, want)


@pytest.mark.parametrize("rows", TWO_TILES)
def test_units_of_two_tiles_share_too(rows):
    test_shared_bounds_change_no_draw(rows, TWO_TILES_V, 0.7, 0.0)


def test_chunks_share_within_their_own_rows():
    rows, V, budget = CHUNKED
    print(f"shared bounds: rows={rows} V={V} budget={budget}", flush=True)
    hidden, w, _ = inputs(rows, V)
    gather = torch.arange(rows, dtype=torch.int32, device=DEV)
    op = binding.MaskOnlyLogits(rows, D, V, max_rows=rows, budget_bytes=budget, device=DEV, sampling=True)
    assert op.plan.num_chunks > 1
    got = drawn(op, hidden, w, gather, gather, 0.7, 41)
    torch.cuda.synchronize()
    check_same(got, drawn_alone(hidden, w, gather, gather, 0.7, 41))


def test_a_hidden_tensor_beyond_4_gib():
    """On the 4-wave kernel, whose units share, and, where the list has a gap of 4 GiB, on the general kernel in its place."""
    T, V, rows = BEYOND_4_GIB
    small, w, _ = inputs(rows, V)
    hidden = torch.empty((T, D), dtype=torch.bfloat16, device=DEV)
    assert T * D * 2 > 1 << 32
    own = torch.arange(rows, dtype=torch.int32, device=DEV)
    want = drawn_alone(small, w, own, own, 0.7, 41)
    for flag, gather in ((0, T - rows + own), (1, torch.where(own < 5, own, T - rows + own))):
        print(f"shared bounds beyond 4 GiB: flag={flag}", flush=True)
        hidden[gather.long()] = small
        op = binding.MaskOnlyLogits(T, D, V, max_rows=rows, device=DEV, sampling=True)
        got = drawn(op, hidden, w, gather.contiguous(), own, 0.7, 41)
        torch.cuda.synchronize()
        assert span_flag(op) == flag
        if flag:                                                    # sums in another order, and with them the scores
            assert (got[0] != want[0]).sum() <= 2 and torch.allclose(got[2], want[2], rtol=1e-6, atol=0)
        else:
            check_same(got, want)
    del hidden
    torch.cuda.empty_cache()


def test_a_drawn_step_as_a_replayed_graph():
    """Captured once and replayed while the mask shrinks, with what an earlier call leaves in the confidences overwritten ahead
    of every replay, against the eager step."""
    T, V = GRAPH
    print(f"drawn graph replay T={T} V={V}", flush=True)
    hidden, w, _ = inputs(T, V)
    seq_starts = torch.tensor([0, T // 3, T], dtype=torch.int32, device=DEV)
    n_per_seq = torch.tensor([T // 9, T // 5], dtype=torch.int32, device=DEV)
    tau, seed, steps = 0.7, 17, 4

    def one_step(op, mask, tokens):
        op.sample_step(hidden, w, mask, tau, seed)
        binding.mosaic_unmask_topn(op.conf, op.token, op.idx, op.count, op.max_rows, seq_starts, n_per_seq, tokens, mask)

    op = binding.MaskOnlyLogits(T, D, V, device=DEV, sampling=True)
    mask, tokens = torch.ones(T, dtype=torch.uint8, device=DEV), torch.full((T,), -1, dtype=torch.int32, device=DEV)
    eager = []
    for _ in range(steps):
        one_step(op, mask, tokens)
        torch.cuda.synchronize()
        n = int(op.count.item())
        eager.append([n] + [x.clone() for x in (op.token[:n], op.conf[:n], op.lse[:n], mask, tokens)])
    assert len({e[0] for e in eager}) == steps
    gop = binding.MaskOnlyLogits(T, D, V, device=DEV, sampling=True)
    gmask, gtokens = torch.ones_like(mask), torch.full_like(tokens, -1)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        one_step(gop, gmask, gtokens)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        one_step(gop, gmask, gtokens)
    torch.cuda.synchronize()
    for _ in range(2):                                              # the whole loop twice
        gmask.fill_(1)
        gtokens.fill_(-1)
        for n, *want in eager:
            gop.conf.fill_(1e30)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert int(gop.count.item()) == n
            for a, b in zip((gop.token[:n], gop.conf[:n], gop.lse[:n], gmask, gtokens), want):
                assert torch.equal(a, b), n
