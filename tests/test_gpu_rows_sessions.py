"""Decode batches of more sessions than a wave has lanes, and than the square of
that: sessions of one length and of very different ones, among them sessions
without keys or without appended tokens, 1, 2 and 4 tokens each, fp8 and MXFP4
keys; against the oracle on every row (row-relative 1e-2, the -inf pattern
exact, nothing written past the scores)."""
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
@pytest.mark.parametrize("N", [1, 2, 4])
@pytest.mark.parametrize("B,even", [(300, False), (300, True), (4100, False)])
def test_sessions(B, even, N, fmt):
    rng = np.random.default_rng(B + N)
    if even:
        hist, new = np.full(B, 700, np.int32), np.full(B, N, np.int32)
    else:
        hist, new = rng.integers(0, 30, B).astype(np.int32), rng.integers(1, N + 1, B).astype(np.int32)
        hist[[1, B // 3, B - 2]] = [3000, 2047, 1100]
        hist[::5], new[3::7], new[0] = 0, 0, N
    wl = make_workload(hist_len=hist, new_len=new, H=64, d=128, idx_dtype="fp8", k=16, seed=B + N, w_scale=0.125,
                       key_format=fmt)
    bt = janus.Batch(wl.hist_len, wl.new_len)
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
        ref = oracle.index_scores_mxfp4(*args, wl.k_bscale, None, wl.w, rows, out_ld=wl.max_ctx)
    else:
        ref = oracle.index_scores(*args, "fp8", wl.k_scale, wl.w, rows, out_ld=wl.max_ctx)
    for b in range(B):
        ctx = int(wl.ctx_len[b])
        for i in range(int(new[b])):
            at = int(wl.score_start[b]) + i * ctx
            got, want = flat[at:at + ctx].astype(np.float64), ref[int(wl.q_start[b]) + i, :ctx]
            fin = np.isfinite(want)
            assert np.array_equal(fin, np.isfinite(got)), (b, i)
            assert np.abs(got[fin] - want[fin]).max() <= 1e-2 * np.abs(want[fin]).max(), (b, i)
