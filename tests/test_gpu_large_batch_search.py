"""Batches of more than 20 000 kept tokens: recovery and assignment in one launch, four tokens per wavefront in the assignment (small
samples whose recovery finds its candidates: one).  Each sample as in a call of its own."""
import numpy as np
import pytest
import torch

import paper_2504_08966_amd as P
from tests import gpu_util as gu
from tests.test_gpu_parity import _random_sample

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("lens,d_h", [([700 + k % 3 for k in range(64)], 8), ([1663 - 61 * (k % 5) for k in range(30)], 64), ([17, 14001, 1, 9000, 14999, 64], 128)])
def test_each_sample_as_in_a_call_of_its_own(lens, d_h, dtype):
    lam, d_c = 0.45, 0.02
    ss = [_random_sample(7700 + k, n, 1, 1, d_h, 64, lam, dtype) for k, n in enumerate(lens)]
    assert sum(n - int(lam * n) for n in lens) > 20000
    hid, ks, qs = (gu.dev(np.concatenate([x(s).reshape(s.n, -1) for s in ss]), dtype) for x in (lambda s: s.hidden, lambda s: s.keys, lambda s: s.queries))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(int)
    prm = [P.PactParams(lam, d_c, 2.0, 1.5) for _ in lens]
    o = P.pact_reduce_varlen(hid, ks, ks, qs, 1, d_h, 1, off.tolist(), prm)
    torch.cuda.synchronize()
    for k in range(0, len(lens), 7 if len(lens) > 8 else 1):
        a, b = off[k], off[k + 1]
        g = P.pact_reduce(hid[a:b], ks[a:b], ks[a:b], qs[a:b], 1, d_h, 1, prm[k])
        torch.cuda.synchronize()
        C = P.read_report(g["rep"])["n_centers"]
        for name, m in (("cluster_id", b - a), ("center_idx", C), ("merged", C), ("cluster_counts", C)):
            assert torch.equal(o[name][a:a + m], g[name][:m]), (k, name)
