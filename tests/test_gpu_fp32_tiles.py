"""Density pass of fp32 keys on both sides of the choice between whole tiles (128 x 128) and halves of them: several turns of either, the last
tile with one token or a few in it, rows that ask for the lowest byte.  Against the oracle, and a batch's samples against calls of their own."""
import numpy as np
import pytest
import torch

import paper_2504_08966_amd as P
from tests import gpu_util as gu
from tests.test_gpu_half_tiles import _check_clustering
from tests.test_gpu_parity import _random_sample

pytestmark = pytest.mark.gpu


# more than one turn of whole tiles: rows of more than 512 elements take those where their last turn is as full as that of the halves (2945, 3457: a last tile of one token; whole
# tiles: the last two), shorter ones halves, 5800 tokens of 64 (eight turns and more) too
@pytest.mark.parametrize("n,dk", [(2945, 520), (3000, 576), (2945, 512), (5800, 64), (5801, 128), (3457, 1032), (3500, 1600)])
def test_clustering(n, dk):
    _check_clustering(n, dk, "f32")


# in turns of the chip: ten of whole tiles and short rows (halves), and 8.2 of 24 slices (whole)
@pytest.mark.parametrize("lens,d_h", [([2500, 2497] * 6, 64), ([2500, 2497] * 5, 1536)])
def test_batch(lens, d_h):
    lam, d_c, H = 0.0, 0.02, 16
    ss = [_random_sample(8100 + k, n, 1, 1, d_h, H, lam, "f32") for k, n in enumerate(lens)]
    hid, ks, qs = (gu.dev(np.concatenate([x(s).reshape(s.n, -1) for s in ss]), "f32") for x in (lambda s: s.hidden, lambda s: s.keys, lambda s: s.queries))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(int)
    prm = [P.PactParams(lam, d_c, 2.0, 1.5) for _ in lens]
    o = P.pact_reduce_varlen(hid, ks, ks, qs, 1, d_h, 1, off.tolist(), prm)
    torch.cuda.synchronize()
    for k in (0, 1, len(lens) - 1):
        a, b = off[k], off[k + 1]
        g = P.pact_reduce(hid[a:b], ks[a:b], ks[a:b], qs[a:b], 1, d_h, 1, prm[k])
        torch.cuda.synchronize()
        C = P.read_report(g["rep"])["n_centers"]
        for name, m in (("cluster_id", b - a), ("center_idx", C), ("merged", C), ("cluster_counts", C)):
            assert torch.equal(o[name][a:a + m], g[name][:m]), (k, name)
