"""Page lists, runs and page demand where their kernels change course,
bit-exact against the oracle: words and slices that end inside a run (pools of
one word to 2^19 pages, one to sixteen blocks), pieces shorter and longer than
a word and the largest max_run, and selections of one launch and of three, with
rows that can and cannot be read 16 bytes at a time."""
import numpy as np
import pytest
import torch

import oracle
from workloads import make_workload, synth_topk

pytestmark = pytest.mark.gpu
janus = pytest.importorskip("paper_2609_36938_amd")


def T(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _pack(bits):
    return np.packbits(bits.reshape(-1, 8), axis=1, bitorder="little").reshape(-1).view(np.uint32)


def _patterns(P):
    n = (P + 31) // 32 * 32
    rng = np.random.default_rng(P)
    at = np.arange(n)
    yield "all", np.ones(n, bool)
    yield "runs", (at // 977) % 3 != 1
    yield "words", (at // 64) % 2 == 0
    yield "dense", rng.random(n) < 0.98
    yield "sparse", rng.random(n) < 0.03


@pytest.mark.parametrize("max_run", [1, 5, 31, 32, 33, 1000, 2 ** 31 - 1])
@pytest.mark.parametrize("P", [1, 31, 64, 1000, 32768, 32769, 70001, 1 << 19])
def test_runs(P, max_run):
    for name, bits in _patterns(P):
        a = _pack(bits)
        a[-1] |= np.uint32(0xffffffff)  # bits past the pool are ignored
        zero = np.zeros_like(a)
        miss, mruns, cnt = janus.predict_diff(T(a.view(np.int32)), T(zero.view(np.int32)), P, max_run)
        torch.cuda.synchronize()
        tail = a.copy()
        if P % 32:
            tail[-1] &= np.uint32((1 << (P % 32)) - 1)
        rmiss, rruns, rcnt = oracle.predict_diff(tail, zero, P, max_run)
        c = cnt.cpu().numpy()
        assert np.array_equal(c, rcnt), (name, c, rcnt)
        assert np.array_equal(miss.cpu().numpy().view(np.uint32), rmiss), name
        assert np.array_equal(mruns.cpu().numpy()[:2 * c[4]].reshape(-1, 2), rruns), name


@pytest.mark.parametrize("k,new,spread", [(30, [5, 3, 2], 1), (64, [5, 0, 9], 1), (64, [5, 1, 9], 40), (512, [20, 11, 2], 1),
                                          (30, [300, 250, 70], 1), (512, [40, 90, 7], 30), (1024, [17, 1, 1], 1)])
def test_page_demand_paths(k, new, spread):
    wl = make_workload(hist_len=[9000, 0, 777], new_len=new, H=2, d=8, idx_dtype="f32", k=k, seed=12, page_size=16)
    sel = synth_topk(wl, seed=4, pad_rows=1)
    P = wl.num_phys_pages * spread + 3
    table = (wl.page_table * spread + 2).astype(np.int32)
    bt = janus.Batch(wl.hist_len, wl.new_len)
    for shift in (0, 1):  # the second copy of the ids is not 16-byte aligned
        ids = torch.zeros(sel.size + 4, dtype=torch.int32, device="cuda")[shift:shift + sel.size].view(sel.shape)
        ids.copy_(T(sel))
        for limit in (None, wl.ctx_len.astype(np.int32)):
            bm, lst, runs, cnt = janus.page_demand(bt, ids, T(table), 16, P, 7,
                                                   limit=None if limit is None else T(limit))
            torch.cuda.synchronize()
            rbm, rlst, rc = oracle.page_demand(wl.q_start, wl.hist_len, sel, table, 16, P, limit=limit)
            rruns = oracle.runs(rbm, P, 7)
            c = cnt.cpu().numpy()
            assert c[0] == rc and c[1] == len(rruns)
            assert np.array_equal(bm.cpu().numpy().view(np.uint32), rbm)
            assert np.array_equal(lst.cpu().numpy()[:rc], rlst)
            assert np.array_equal(runs.cpu().numpy()[:2 * c[1]].reshape(-1, 2), rruns)
