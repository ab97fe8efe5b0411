"""Recovery where every centre is a candidate (pruned keys of norm zero within a threshold above 1): the rows that fill up the last
group of 64 centres are not."""
import numpy as np
import pytest
import torch

import paper_2504_08966_amd as P
from tests import gpu_util as gu
from tests.test_gpu_parity import _random_sample, assert_same, oracle_reduce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,d_h", [(20, 64), (300, 64), (300, 512), (3000, 64)])
def test_zero_vectors_within_reach_of_all_centres(n, d_h, dtype):
    s = _random_sample(7300 + n, n, 1, 1, d_h, 64, 0.5, dtype)
    zero = np.arange(1, n, 5)
    s.keys[zero] = 0.0
    s.hidden[zero] *= 2.0 ** -20                                     # (pruned)
    o = oracle_reduce(s, 0.8)
    assert len(o["center_idx"]) % 64 and np.isin(zero, o["pruned_idx"]).all()
    assert (o["cluster_id"][zero] >= 0).all()                        # distance 1, threshold 1.2
    hid, ks, qs = (gu.dev(x.reshape(n, -1), dtype) for x in (s.hidden, s.keys, s.queries))
    g = P.pact_reduce(hid, ks, ks, qs, 1, d_h, 1, P.PactParams(0.5, 0.8, 2.0, 1.5))
    torch.cuda.synchronize()
    assert_same(gu.trim(g, n), o, s, f"n={n} d_h={d_h} {dtype}")
