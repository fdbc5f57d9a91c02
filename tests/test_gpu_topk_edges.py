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
