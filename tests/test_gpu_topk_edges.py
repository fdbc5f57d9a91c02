"""Top-k where its kernel changes course, exact against the oracle's full sort:
rows one candidate longer than k, at and past the buffer sizes (4096 and 8192
entries: no seed and a seed), odd context lengths (rows that do not start on
16 bytes), the largest k, contexts past the small kernel's bitmap, and fills
that overflow the buffer in every order, tie the whole row, or hold few
distinct values."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_parity import FILLS

pytestmark = pytest.mark.gpu
janus = pytest.importorskip("paper_2609_36938_amd")

SIZES = [(1, 1, 1), (64, 2, 64), (2048, 3, 2048), (4094, 4, 2048), (4099, 2, 100), (8190, 4, 6144), (9001, 3, 6144),
         (16383, 2, 2047), (40000, 2, 4000), (262200, 1, 2048)]


# (the longest row: one order, one tie-heavy and one usual fill)
CASES = [(f, *s) for s in SIZES for f in FILLS if s[0] < 200000 or f in ("hot", "descending", "few_levels")]


@pytest.mark.parametrize("fill,hist,new,k", CASES)
def test_topk_edges(fill, hist, new, k):
    rng = np.random.default_rng(7)
    ctx = hist + new
    rows = np.full((new, ctx), -np.inf, np.float32)
    for i in range(new):
        rows[i, :hist + i + 1] = FILLS[fill](rng, 0, i, hist + i + 1)
    bt = janus.Batch([hist], [new])
    sel = janus.topk(bt, torch.from_numpy(rows.reshape(-1)).cuda(), k)
    torch.cuda.synchronize()
    got = sel.cpu().numpy()
    ref = oracle.topk([0, new], [hist], np.arange(new), rows, k)
    for i in range(new):
        want = min(k, hist + i + 1)
        assert np.all(got[i, want:] == -1) and np.all(np.diff(got[i, :want]) > 0)
        assert np.array_equal(got[i, :want], np.sort(ref[i, :want])), (fill, i)


@pytest.mark.parametrize("ctx,k", [(5000, 2048), (40000, 1000), (131072, 2048), (131072, 2)])
@pytest.mark.parametrize("levels", [1, 2, 50])
def test_ties_below_outliers(ctx, k, levels):
    """Few scores far above the rest, which lie on one or some neighbouring values: the first
    range narrowing puts them into one bin, the next ones onto one bin again or side by side."""
    rng = np.random.default_rng(ctx + levels)
    row = (1 + rng.integers(0, levels, ctx) * 2.0 ** -23).astype(np.float32)
    high = rng.random(ctx) < 0.002
    row[high] = 10.0 ** rng.uniform(1, 30, int(high.sum()))
    bt = janus.Batch([ctx - 1], [1])
    sel = janus.topk(bt, torch.from_numpy(row).cuda(), k)
    torch.cuda.synchronize()
    ref = oracle.topk([0, 1], [ctx - 1], [0], row[None], k)
    assert np.array_equal(sel.cpu().numpy(), np.sort(ref, axis=1))


def _sampled(row):
    """The scores of the seed's sample in a 16-byte aligned row: 512 groups of 8 spread over it."""
    ng = len(row) >> 3
    g = np.arange(512) * ng // 512
    return (8 * g[:, None] + np.arange(8)).reshape(-1)


def _passes(row, k, seed):
    """Fewest and most elements that a threshold from the sample can let through: the lower
    end of a narrow range of values around the sample's rank."""
    s = np.sort(row[_sampled(row)])[::-1]
    r = int(np.float32(seed) * k * len(s) / len(row)) + 8
    return int((row >= s[r - 1]).sum()), int((row >= s[min(len(s), r + max(4, r >> 3) + 1) - 1]).sum())


@pytest.mark.parametrize("k", [1000, 2048])
@pytest.mark.parametrize("ctx", [40000, 131072, 262400])
@pytest.mark.parametrize("misses", [1, 2])
def test_seed_misses(ctx, misses, k):
    """High scores exactly in the sample, too few to fill k: the first threshold (misses = 1) or
    the looser second one too (misses = 2) lies above the k-th score, and the row is streamed again."""
    new = 4
    rng = np.random.default_rng(ctx + k)
    rows = np.full((new, ctx), -np.inf, np.float32)
    for i in range(new):
        n = ctx - new + i + 1
        rows[i, :n] = rng.random(n)
        at = _sampled(rows[i, :n])
        h = int((1.25 if misses == 1 else 3.5) * 1.3 * k * len(at) / n) + 12 * misses
        assert h < k
        rows[i, rng.choice(at, h, replace=False)] += 10
        lo, hi = _passes(rows[i, :n], k, 1.3)
        assert hi < k
        lo, hi = _passes(rows[i, :n], k, 3.0)
        assert hi < k if misses == 2 else k <= lo
    bt = janus.Batch([ctx - new], [new])
    sel = janus.topk(bt, torch.from_numpy(rows.reshape(-1)).cuda(), k)
    torch.cuda.synchronize()
    ref = oracle.topk([0, new], [ctx - new], np.arange(new), rows, k)
    assert np.array_equal(sel.cpu().numpy(), np.sort(ref, axis=1))
