"""Prefill indexer scores of sessions whose contexts differ by three orders of
magnitude: every session is cut into the same number of key chunks (16 here,
the longest session being past 131072 keys), so that the short ones have
chunks of a single stage, part of one, or none.  fp8, bf16 and MXFP4 keys, and
entries, against the oracle on every row: the causal -inf pattern exactly and,
per row, max |gpu - oracle| / max |oracle| <= 1e-2 (bf16 1e-3)."""
import numpy as np
import pytest
import torch

import oracle
from workloads import make_workload

pytestmark = pytest.mark.gpu
janus = pytest.importorskip("paper_2609_36938_amd")


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("keys,es", [("fp8", 0), ("bf16", 0), ("mxfp4", 0), ("fp8", 2)])
def test_ragged_chunks(keys, es):
    hist, new = [132000 << es, 129 << es, 0, 2047 << es, 5000 << es], [6, 5, 7, 9, 13]
    wl = make_workload(hist_len=hist, new_len=new, H=64, d=128, idx_dtype="bf16" if keys == "bf16" else "fp8", k=64,
                       seed=91, w_scale=0.125, key_format="mxfp4" if keys == "mxfp4" else None, entry_shift=es)
    bt = janus.Batch(wl.hist_len, wl.new_len, entry_shift=es)
    q, kI, w = T(wl.q), T(wl.kI), T(wl.w)
    sq = None if wl.q_scale is None else T(wl.q_scale)
    if keys == "mxfp4":
        sc = janus.index_scores_mxfp4(bt, q, kI, T(wl.k_bscale), w, q_scale=sq)
    else:
        sc = janus.index_scores(bt, q, kI, w, q_scale=sq, k_scale=None if wl.k_scale is None else T(wl.k_scale),
                                dtype=keys)
    torch.cuda.synchronize()
    flat = sc.cpu().numpy()
    rows = np.arange(wl.total_q)
    if keys == "mxfp4":
        ref = oracle.index_scores_mxfp4(wl.q_start, wl.hist_len, wl.q, "fp8", wl.q_scale, wl.kI, wl.k_bscale, None,
                                        wl.w, rows, out_ld=wl.max_ctx)
    else:
        ref = oracle.index_scores(wl.q_start, wl.hist_len, wl.q, keys, wl.q_scale, wl.kI, keys, wl.k_scale, wl.w,
                                  rows, out_ld=wl.max_ctx, entry=1 << es)
    tol = 1e-3 if keys == "bf16" else 1e-2
    for b in range(wl.num_seqs):
        ctx = int(wl.ctx_len[b])
        for i in range(int(wl.new_len[b])):
            at = int(wl.score_start[b]) + i * ctx
            got, want = flat[at:at + ctx].astype(np.float64), ref[int(wl.q_start[b]) + i, :ctx]
            fin = np.isfinite(want)
            assert np.array_equal(fin, np.isfinite(got)), (b, i)
            if fin.any():
                assert np.abs(got[fin] - want[fin]).max() <= tol * np.abs(want[fin]).max(), (b, i)
