"""Compaction and top-n unmasking at the sizes where their paths meet: sequences around the row count up to which rows are ranked
directly, none, one and all rows taken, sequence lengths around the block's 1024 threads, many exact ties, a
confidence of zero.  Bit-exact against the oracle."""
import numpy as np
import pytest
import torch

from paper_2601_06562_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("rows", [1, 3, 63, 64, 255, 256, 257, 1023, 1024, 1025, 5000])
@pytest.mark.parametrize("levels", [2, 0])
def test_sequences_around_the_path_boundaries(rows, levels):
    import oracle
    print(f"unmask edges rows={rows} levels={levels}", flush=True)
    rng = np.random.default_rng(rows + levels)
    per_seq = [rows, 0, max(1, rows // 2), rows]                 # masked rows of four sequences, gaps between them
    starts, pos, t = [0], [], 0
    for n in per_seq:
        span = 2 * n + 5
        pos.append(t + np.sort(rng.choice(span, n, replace=False)))
        t += span
        starts.append(t)
    idx = np.concatenate(pos).astype(np.int32)
    seq_starts = np.array(starts, np.int32)
    mask = np.zeros(t, np.uint8)
    mask[idx] = 1
    conf = (rng.choice(np.array([0.0, 0.25], np.float32), idx.size) if levels
            else np.exp2(-12 * rng.random(idx.size)).astype(np.float32))
    tok = rng.integers(0, 150000, idx.size).astype(np.int32)
    tokens = rng.integers(0, 150000, t).astype(np.int32)
    dev = lambda a, dt: torch.as_tensor(a, dtype=dt, device=DEV)
    for n_per_seq in ([1, 1, 0, rows], [rows // 2, 3, 1, rows + 7], [rows - 1, 0, rows, 2]):
        n_per_seq = np.array(n_per_seq, np.int32)
        want_tokens, want_mask, _ = oracle.unmask_topn(conf, tok, idx, seq_starts, n_per_seq, tokens, mask)
        d_tokens, d_mask = dev(tokens, torch.int32), dev(mask, torch.uint8)
        binding.mosaic_unmask_topn(dev(conf, torch.float32), dev(tok, torch.int32), dev(idx, torch.int32),
                                   dev([idx.size], torch.int32), idx.size, dev(seq_starts, torch.int32),
                                   dev(n_per_seq, torch.int32), d_tokens, d_mask)
        torch.cuda.synchronize()
        assert np.array_equal(d_mask.cpu().numpy(), want_mask), n_per_seq
        assert np.array_equal(d_tokens.cpu().numpy(), want_tokens), n_per_seq


@pytest.mark.parametrize("T", [65536, 65537, 69632, 1024 * 4096, 1024 * 4096 + 1])
def test_compaction_where_its_paths_meet(T):
    """One block up to 65536 positions; then blocks that add up the counts before them themselves; from 1024 blocks of
    4096 positions on, a scan of the counts."""
    print(f"compaction edges T={T}", flush=True)
    rng = np.random.default_rng(T)
    for p in (0.0, 0.001, 0.6):
        mask = (rng.random(T) < p).astype(np.uint8)
        mask[[0, T - 1]] = 1 if p else 0
        want = np.nonzero(mask)[0].astype(np.int32)
        d_mask = torch.as_tensor(mask, device=DEV)
        idx = torch.full((T,), -7, dtype=torch.int32, device=DEV)
        count = torch.full((1,), -7, dtype=torch.int32, device=DEV)
        scratch = torch.empty(binding.mosaic_compact_scratch_bytes(T), dtype=torch.uint8, device=DEV)
        binding.mosaic_mask_compact(d_mask, idx, count, scratch)
        torch.cuda.synchronize()
        got = idx.cpu().numpy()
        assert int(count.item()) == want.size
        assert np.array_equal(got[:want.size], want) and np.all(got[want.size:] == -7)
