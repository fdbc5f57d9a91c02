"""A page table entry past the pool, but within the bitmap's last word, is kept
out of the page list, the runs and the counts by one launch as by three."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
janus = pytest.importorskip("paper_2609_36938_amd")


@pytest.mark.parametrize("rows", [2, 40])  # one launch, three
def test_entries_past_the_pool(rows):
    P = 33  # bits 33 .. 63 of the second word stand for no page
    table = torch.tensor([[3, 4, 32, 33, 60, 63]], dtype=torch.int32, device="cuda")
    bt = janus.Batch([6 * 16], [rows])
    pages = 6 + -(-rows // 16)
    table = torch.nn.functional.pad(table, (0, pages - 6))
    ids = torch.arange(0, 96, 16, dtype=torch.int32, device="cuda").repeat(rows, 1).contiguous()
    out = tuple(torch.full((n,), -7, dtype=torch.int32, device="cuda") for n in (2, P + 40, 2 * P + 80, 2))
    bm, lst, runs, cnt = janus.page_demand(bt, ids, table, 16, P, 32, out=out)
    torch.cuda.synchronize()
    assert cnt.tolist() == [3, 2] and lst.tolist()[:4] == [3, 4, 32, -7] and runs.tolist()[:5] == [3, 2, 32, 1, -7]
    assert (bm.cpu().numpy().view(np.uint32)[0] >> 3) & 3 == 3
