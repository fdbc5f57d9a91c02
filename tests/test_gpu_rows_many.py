"""Decode batches of one token per session whose blocks are numbered through
the sessions' chunk counts, 64 sessions at a time: batches of 1, 64, 65 and 200
sessions, contexts from one key to many chunks, sessions that append nothing,
entries; fp8 and MXFP4 keys, against the oracle on every row (row-relative
1e-2, the -inf pattern exact)."""
import numpy as np
import pytest
import torch

import oracle
from workloads import make_workload

pytestmark = pytest.mark.gpu
janus = pytest.importorskip("paper_2609_36938_amd")


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("fmt", [None, "mxfp4"])
@pytest.mark.parametrize("B,es", [(1, 0), (64, 0), (65, 0), (200, 0), (70, 2)])
def test_many_sessions(B, es, fmt):
    rng = np.random.default_rng(B)
    hist = (rng.integers(0, 1500, B) << es).astype(np.int32)
    hist[::7] = 0
    hist[B // 2] = 5000 << es
    new = np.ones(B, np.int32)
    new[3::5] = 0
    wl = make_workload(hist_len=hist, new_len=new, H=64, d=128, idx_dtype="fp8", k=16, seed=B + 1, w_scale=0.125,
                       key_format=fmt, entry_shift=es)
    bt = janus.Batch(wl.hist_len, wl.new_len, entry_shift=es)
    sc = torch.full((bt.total_scores + 4,), 3.0, device="cuda")
    if fmt:
        janus.index_scores_mxfp4(bt, T(wl.q), T(wl.kI), T(wl.k_bscale), T(wl.w), q_scale=T(wl.q_scale),
                                 scores=sc[:bt.total_scores])
    else:
        janus.index_scores(bt, T(wl.q), T(wl.kI), T(wl.w), q_scale=T(wl.q_scale), k_scale=T(wl.k_scale),
                           scores=sc[:bt.total_scores])
    torch.cuda.synchronize()
    assert bool((sc[bt.total_scores:] == 3).all())
    flat = sc.cpu().numpy()
    rows = np.arange(wl.total_q)
    args = (wl.q_start, wl.hist_len, wl.q, "fp8", wl.q_scale, wl.kI)
    if fmt:
        ref = oracle.index_scores_mxfp4(*args, wl.k_bscale, None, wl.w, rows, out_ld=wl.max_ctx, entry=1 << es)
    else:
        ref = oracle.index_scores(*args, "fp8", wl.k_scale, wl.w, rows, out_ld=wl.max_ctx, entry=1 << es)
    for b in range(B):
        if new[b] == 0 or wl.ctx_len[b] == 0:
            continue
        at, ctx = int(wl.score_start[b]), int(wl.ctx_len[b])
        got, want = flat[at:at + ctx].astype(np.float64), ref[int(wl.q_start[b]), :ctx]
        fin = np.isfinite(want)
        assert np.array_equal(fin, np.isfinite(got)), b
        if fin.any():
            assert np.abs(got[fin] - want[fin]).max() <= 1e-2 * np.abs(want[fin]).max(), b
