"""Indexer scores (Eq. 1) of the shapes and dtypes that have no kernel of their
own (index_scores_general), against the oracle on every row.

Cases sit where its tiles end: heads that are no multiple of 4, fill a block's
64 rows or run past them, dims that are no multiple of 4 or 16 or run past the
64 staged at a time, key and query rows without 16-byte alignment, a ragged
batch with an empty history, entries.  Compared: the causal -inf pattern
exactly and, per row, max |gpu - oracle| / max |oracle| <= 1e-5 (fp32; sums of
up to 64 x 130 fp32 terms), 1e-3 (bf16), 1e-2 (fp8: the stated tolerances)."""
import numpy as np
import pytest
import torch

import oracle
from workloads import make_workload

pytestmark = pytest.mark.gpu
janus = pytest.importorskip("paper_2609_36938_amd")

TOL = {"f32": 1e-5, "bf16": 1e-3, "fp8": 1e-2}


def _shifted(a, shift):
    """The array on the GPU, `shift` elements past an aligned address."""
    t = torch.from_numpy(np.ascontiguousarray(a))
    out = torch.zeros(t.numel() + 16, dtype=t.dtype, device="cuda")[shift:shift + t.numel()].view(t.shape)
    return out.copy_(t)


@pytest.mark.parametrize("dt,H,d,shift,es", [
    ("f32", 1, 1, 0, 0), ("f32", 4, 64, 0, 0), ("f32", 4, 64, 1, 0), ("f32", 3, 50, 0, 0), ("f32", 70, 130, 0, 0),
    ("f32", 12, 68, 0, 3), ("f32", 64, 128, 0, 0), ("f32", 130, 16, 0, 0), ("bf16", 16, 32, 0, 0),
    ("bf16", 64, 96, 1, 0), ("bf16", 5, 20, 0, 2), ("fp8", 8, 24, 0, 0), ("fp8", 64, 64, 3, 0), ("fp8", 33, 129, 0, 0)])
def test_general_shapes(dt, H, d, shift, es):
    wl = make_workload(hist_len=[300, 0, 65], new_len=[19, 9, 66], H=H, d=d, idx_dtype=dt, k=16, seed=41,
                       w_scale=0.125, entry_shift=es)
    bt = janus.Batch(wl.hist_len, wl.new_len, entry_shift=es)
    sc = torch.full((bt.total_scores + 8,), 5.0, device="cuda")
    scale = {} if wl.q_scale is None else {"q_scale": _shifted(wl.q_scale, 0), "k_scale": _shifted(wl.k_scale, 0)}
    janus.index_scores(bt, _shifted(wl.q, shift), _shifted(wl.kI, shift), _shifted(wl.w, 0), dtype=dt,
                       scores=sc[:bt.total_scores], **scale)
    torch.cuda.synchronize()
    assert bool((sc[bt.total_scores:] == 5).all())
    flat = sc[:bt.total_scores].cpu().numpy()
    rows = np.arange(wl.total_q)
    ref = oracle.index_scores(wl.q_start, wl.hist_len, wl.q, dt, wl.q_scale, wl.kI, dt, wl.k_scale, wl.w, rows,
                              out_ld=max(1, wl.max_ctx), entry=1 << es)
    for b in range(wl.num_seqs):
        ctx = int(wl.ctx_len[b])
        for i in range(int(wl.new_len[b])):
            at = int(wl.score_start[b]) + i * ctx
            got, want = flat[at:at + ctx].astype(np.float64), ref[int(wl.q_start[b]) + i, :ctx]
            fin = np.isfinite(want)
            assert np.array_equal(fin, np.isfinite(got)), (b, i)
            if fin.any():
                assert np.abs(got[fin] - want[fin]).max() <= TOL[dt] * np.abs(want[fin]).max(), (b, i)


def test_general_keeps_subnormal_products():
    """Products below the smallest normal fp32 are not flushed to zero."""
    bt = janus.Batch([40], [2])
    q = torch.full((2, 4, 64), 1e-20, device="cuda")
    kI = torch.full((42, 64), 1e-20, device="cuda")
    sc = janus.index_scores(bt, q, kI, torch.ones((2, 4), device="cuda"))
    torch.cuda.synchronize()
    got = sc.cpu().numpy().reshape(2, 42)[1].astype(np.float64)
    assert np.all(np.abs(got / (4 * 64 * np.float64(np.float32(1e-20)) ** 2) - 1) < 1e-4)
