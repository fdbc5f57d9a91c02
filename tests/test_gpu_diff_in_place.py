"""janus_predict_diff with the miss set written over one of its inputs: pools
whose runs one block emits and pools that take several, bit-exact against the
oracle on the inputs as they were."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
janus = pytest.importorskip("paper_2609_36938_amd")


@pytest.mark.parametrize("over", ["actual", "predicted"])
@pytest.mark.parametrize("P", [33, 32768, 32769, 70001, 1 << 19])
def test_in_place(P, over):
    nw = (P + 31) // 32
    rng = np.random.default_rng(P)
    for dens in (0.03, 0.5, 0.98):
        a, p = (np.packbits(rng.random(nw * 32) < dens).view(np.uint32) for _ in range(2))
        da, dp = (torch.from_numpy(x.view(np.int32)).cuda() for x in (a, p))
        out = (da if over == "actual" else dp, torch.empty(2 * P, dtype=torch.int32, device="cuda"),
               torch.empty(5, dtype=torch.int32, device="cuda"))
        miss, runs, cnt = janus.predict_diff(da, dp, P, 7, out=out)
        torch.cuda.synchronize()
        if P % 32:
            a[-1] &= np.uint32((1 << (P % 32)) - 1)
            p[-1] &= np.uint32((1 << (P % 32)) - 1)
        rmiss, rruns, rcnt = oracle.predict_diff(a, p, P, 7)
        c = cnt.cpu().numpy()
        assert np.array_equal(c, rcnt)
        assert np.array_equal(miss.cpu().numpy().view(np.uint32), rmiss)
        assert np.array_equal(runs.cpu().numpy()[:2 * c[4]].reshape(-1, 2), rruns)
