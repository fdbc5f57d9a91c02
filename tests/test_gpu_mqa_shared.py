"""MQA attention (dqk = dv = 128) on both sides of the rule by which a block's
four waves share one token (few tokens, long selections), against the oracle:
no more tiles than waves, a ragged last tile, rows without a valid id, outputs
without 16-byte alignment.  2e-2 absolute and of the largest
output, lse to 2e-3; a logit scale that moves the running max in later tiles."""
import numpy as np
import pytest
import torch

import oracle
from workloads import attention_inputs, make_workload, synth_topk

pytestmark = pytest.mark.gpu
janus = pytest.importorskip("paper_2609_36938_amd")


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("Hq,k,new,scale", [(8, 256, [256], 0.088), (1, 1, [3, 2], 0.088), (16, 31, [5, 1], 1.0),
                                            (5, 129, [9], 1.0), (8, 128, [4], 1.0), (16, 1024, [6, 250], 1.0),
                                            (8, 129, [257], 1.0), (16, 300, [800, 220], 1.0), (3, 700, [200, 61], 0.088)])
def test_mqa(Hq, k, new, scale):
    attn = dict(Hq=Hq, dqk=128, dv=128, mla=False, q_std=1.0, kv_std=1.0, scale=scale)
    wl = make_workload(hist_len=[1800, 100][:len(new)], new_len=new, H=2, d=8, idx_dtype="f32", k=k, seed=21 + Hq,
                       table="permuted", attn=attn)
    ai, sel = attention_inputs(wl), synth_topk(wl, seed=5, pad_rows=2)
    if wl.total_q > 3:
        sel[1, :] = -1
    bt = janus.Batch(wl.hist_len, wl.new_len)
    n = wl.total_q * Hq * 128
    out = torch.full((n + 8,), 7.0, device="cuda")
    _, lse = janus.sparse_attn(bt, T(ai.q), T(ai.k_pool), T(ai.v_pool), T(wl.page_table), wl.page_size, T(sel),
                               ai.scale, dv=128, out_dtype="f32", want_lse=True, out=out[1:n + 1])
    torch.cuda.synchronize()
    assert float(out[0]) == 7 and bool((out[n + 1:] == 7).all())
    got, gl = out[1:n + 1].cpu().numpy().reshape(wl.total_q, Hq, 128), lse.cpu().numpy()
    rows = np.arange(wl.total_q)
    ref, lref = oracle.sparse_attn(wl.q_start, wl.hist_len, rows, ai.q, ai.k_pool, ai.v_pool, ai.k_row_stride,
                                   ai.v_row_stride, wl.page_table, wl.page_size, sel, ai.scale, ai.dv)
    assert np.abs(got - ref).max() <= 2e-2 * max(1.0, np.abs(ref).max())
    fin = np.isfinite(lref)
    assert np.array_equal(fin, np.isfinite(gl)) and np.all(got[~fin] == 0)
    assert np.allclose(gl[fin], lref[fin], atol=2e-3, rtol=1e-4)
