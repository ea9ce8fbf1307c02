"""The measured cases: what a user of this library has it do, through the public entry points of the binding.

A case is one denoising step of a diffusion language model (compaction of the mask, mask-only logits with the
vocabulary reduction, greedy or by temperature sampling, optionally with the shifted gather list), or, with "steps" > 0,
the tail of several such steps (each followed by top-n unmasking, the plan renewed for the masks that remain, as
``paper_2601_06562_amd/example.py`` does).  Fields of a case:

  batch, length   sequences and positions of each; they are concatenated (T = batch * length)
  d, vocab        hidden size and vocabulary size
  tail, ratio     masked positions: a share `ratio` of the last `tail` positions of every sequence
                  (tail = length: anywhere); ratio < 0: the eight per-sequence ratios of the batched workload
  temperature     0 = greedy
  shift           True: position p is predicted from hidden row p - 1 (the noise stays keyed by p)
  steps           0 = one step, its outputs; n = a tail of n steps, the token sequence and the mask it leaves
  loose           True: the object is made with its default bound on the masked rows (all T positions), as a program
                  does that does not count its masks or replays one captured step; False: with the number of masks
  budget          byte budget of the chunk selector, 0 = unbounded
"""
from __future__ import annotations

import math

import torch

from paper_2601_06562_amd import MaskOnlyLogits, binding
from paper_2601_06562_amd.workloads import BATCHED_RATIOS

DEVICE = "cuda:0"


def _case(name=None, *, batch=1, length, d=4096, vocab=126464, tail=None, ratio=1.0, temperature=0.0, shift=False,
          steps=0, loose=False, budget=0):
    c = {} if name is None else {"name": name}
    c.update(batch=batch, length=length, d=d, vocab=vocab, tail=length if tail is None else tail, ratio=ratio,
             temperature=temperature, shift=shift, steps=steps, loose=loose, budget=budget)
    return c


def listed():
    return [
        # The smallest call: the first benchmark configuration with the object's default arguments.
        _case("tiny", length=512, d=512, vocab=8192, ratio=0.5234, loose=True),
        # Block-wise decoding: a block of 32 positions behind a prompt, emptied in four steps of eight tokens.
        _case("block_32", length=4096, tail=32, steps=4),
        # The last steps of a longer block: about 200 masked positions of the last 512 (the benchmark's few-rows case).
        _case("block_tail", length=4096, tail=512, ratio=0.4),
        # A served batch of eight sequences, each inside a block of 64 positions, drawn at a temperature.
        _case("batch_blocks", batch=8, length=1000, tail=64, ratio=0.55, temperature=0.7),
        # The middle of a denoising run with one plan for the whole run.
        _case("half_masked", length=4096, ratio=0.507, loose=True),
        # A vocabulary that is no multiple of the tile, and an ordinary number of rows.
        _case("ragged_vocab", length=8191, d=3584, vocab=151936, ratio=0.12),
        # A very long context (hidden states beyond 4 GiB), the last block half done, as a tail of two steps.
        _case("long_context", length=600000, tail=2048, ratio=0.49, steps=2),
        # The benchmark's headline: the first step of a 4096-token generation, everything masked.
        _case("first_step", length=4096),
        # The same under temperature sampling.
        _case("first_step_sampled", length=4096, temperature=1.0),
        # Semi-autoregressive decoding behind a long prompt.
        _case("semi_ar", length=32768, tail=8192, ratio=0.5011),
        # A late step of a shifted-prediction model at temperature 0.7.
        _case("late_step_shifted", length=65536, d=3584, vocab=152064, ratio=0.1, temperature=0.7, shift=True),
        # A batch of eight sequences at different stages, one step with its unmasking.
        _case("batched_mixed", batch=8, length=16384, ratio=-1.0, steps=1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    d, vocab = rng.choice([(512, 8192), (1024, 32000), (2048, 65536), (3584, 152064), (3584, 151936), (4096, 126464),
                           (4096, 126464), (4096, 126349)])
    batch = rng.choice([1, 1, 1, 2, 3, 8])
    rows = _log_int(rng, 24, 16384)                                  # masked positions, about
    per_seq = max(1, rows // batch)
    ratio = rng.choice([1.0, 0.75, 0.5, 0.3, 0.1])
    tail = max(8, int(per_seq / ratio))
    length = min(131072 // batch, tail + _log_int(rng, 16, 65536))    # a prompt in front of the block
    if rng.random() < 0.25:
        tail = length                                                # masks anywhere
        ratio = min(1.0, per_seq / length)
    tail = min(tail, length)
    return _case(batch=batch, length=length, d=d, vocab=vocab, tail=tail, ratio=ratio,
                 temperature=rng.choice([0.0, 0.0, 0.0, 0.5, 1.0]), shift=rng.random() < 0.2,
                 steps=rng.choice([0, 0, 1, 3]), loose=rng.random() < 0.25,
                 budget=rng.choice([0, 0, 0, 0, 0, 4 << 20]))


def _rows(case):
    """Masked positions of every sequence."""
    B, tail = case["batch"], case["tail"]
    ratios = [BATCHED_RATIOS[b % 8] if case["ratio"] < 0 else case["ratio"] for b in range(B)]
    return [max(1, min(tail, round(tail * r))) for r in ratios]


def _mask(case, gen):
    """Per sequence a fixed number of masked positions, at places drawn among its last `tail`."""
    B, L, tail = case["batch"], case["length"], case["tail"]
    mask = torch.zeros((B, L), dtype=torch.uint8, device=DEVICE)
    order = torch.rand((B, tail), generator=gen, device=DEVICE).argsort(dim=1)
    for b, n in enumerate(_rows(case)):
        mask[b, L - tail + order[b, :n]] = 1
    return mask


class _State:
    pass


def prepare(case, seed):
    """Inputs on the GPU: LM head N(0, 1/d); hidden rows N(0, 1) plus a multiple (0 to 24) of one LM-head row each, so
    that the predictions range from flat to certain as a model's do; the library object with its plan and buffers."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    s = _State()
    B, L, d, V = case["batch"], case["length"], case["d"], case["vocab"]
    T = B * L
    s.w = torch.empty((V, d), dtype=torch.bfloat16, device=DEVICE)
    for r in range(0, V, 16384):
        n = min(V, r + 16384) - r
        s.w[r:r + n] = torch.randn((n, d), generator=gen, device=DEVICE) * d ** -0.5
    s.hidden = torch.empty((T, d), dtype=torch.bfloat16, device=DEVICE)
    for r in range(0, T, 16384):
        n = min(T, r + 16384) - r
        target = torch.randint(0, V, (n,), generator=gen, device=DEVICE)
        pull = 24.0 * torch.rand((n, 1), generator=gen, device=DEVICE)
        s.hidden[r:r + n] = torch.randn((n, d), generator=gen, device=DEVICE).add_(pull * s.w[target])
    mask = _mask(case, gen)
    s.per_seq = _rows(case)                                          # the scheduler knows its masks
    s.mask = mask.reshape(T)
    s.tokens = torch.randint(0, V, (T,), generator=gen, device=DEVICE, dtype=torch.int32)
    s.seq_starts = torch.tensor([b * L for b in range(B + 1)], dtype=torch.int32, device=DEVICE)
    s.M, s.T, s.steps = sum(s.per_seq), T, case["steps"]
    s.n_step = [-(-m // s.steps) for m in s.per_seq] if s.steps else []
    s.n_per_seq = torch.tensor(s.n_step or [0], dtype=torch.int32, device=DEVICE)
    s.temperature, s.shift, s.loose, s.budget = case["temperature"], case["shift"], case["loose"], case["budget"]
    s.seed = 1000 + int(seed)
    s.op = MaskOnlyLogits(T, d, V, max_rows=None if s.loose else s.M, budget_bytes=s.budget, device=DEVICE,
                          sampling=s.temperature > 0)
    s.gather = torch.empty(T, dtype=torch.int32, device=DEVICE) if s.shift else None
    return s


def _step(s, mask, seed):
    op = s.op
    if s.shift:
        binding.mosaic_mask_compact(mask, op.idx, op.count, op.scratch)
        binding.mosaic_shift_indices(op.idx, op.count, op.max_rows, s.seq_starts, s.gather)
        if s.temperature > 0:
            binding.mosaic_masked_logits_sample(s.hidden, s.w, s.gather, op.count, op.max_rows, s.temperature, seed,
                                                op.token, op.conf, op.lse, op.plan, op.workspace, noise_idx=op.idx)
        else:
            binding.mosaic_masked_logits_reduce(s.hidden, s.w, s.gather, op.count, op.max_rows, op.token, op.conf,
                                                op.lse, op.plan, op.workspace)
    elif s.temperature > 0:
        op.sample_step(s.hidden, s.w, mask, s.temperature, seed)
    else:
        op.step(s.hidden, s.w, mask)


def run(s):
    op = s.op
    if not s.steps:
        _step(s, s.mask, s.seed)
        return {"idx": op.idx[:s.M], "count": op.count, "token": op.token[:s.M], "conf": op.conf[:s.M],
                "lse": op.lse[:s.M]}
    tokens, mask = s.tokens.clone(), s.mask.clone()
    for k in range(s.steps):
        remaining = sum(max(0, m - k * n) for m, n in zip(s.per_seq, s.n_step))
        if not s.loose:
            op.replan(remaining, s.budget)
        _step(s, mask, s.seed + k)
        binding.mosaic_unmask_topn(op.conf, op.token, op.idx, op.count, op.max_rows, s.seq_starts, s.n_per_seq, tokens,
                                   mask)
    n = remaining                                                    # rows of the last step
    return {"tokens": tokens, "mask": mask, "conf": op.conf[:n], "lse": op.lse[:n]}


def work(case):
    """Per step: the mask, the masked hidden rows and the LM head read once, the list and three results per row
    written; 2 flops per row, hidden unit and vocabulary id."""
    B, L, d, V = case["batch"], case["length"], case["d"], case["vocab"]
    per_seq = _rows(case)
    steps = max(1, case["steps"])
    total = {"bytes": 0.0, "flops": 0.0}
    for k in range(steps):
        rows = sum(max(0, m - k * -(-m // steps)) for m in per_seq)
        total["bytes"] += 2.0 * V * d + 2.0 * rows * d + B * L + 16.0 * rows
        total["flops"] += 2.0 * rows * d * V
    if case["steps"]:
        total["bytes"] += 5.0 * B * L + 5.0 * sum(per_seq)           # the token sequence and the mask written
    return total


def tolerance(case):
    """Exact products, 32-bit sums, hardware exponentials.  The fused pass against the same pass on the general kernel,
    whose sums run in another order, measured over the single-step cases: conf and lse off by at most 3.3e-7 (2-norm)
    and 2.3e-6 (largest), every id equal; about four times that.  Ids may differ where two scores tie within rounding,
    and so may the positions at the edge of a top n."""
    return {"rel": 2e-6, "max": 1e-5, "differ": 1e-3}
