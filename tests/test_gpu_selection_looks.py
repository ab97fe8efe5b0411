"""Centre selection of samples above 1024 tokens: statuses joined by OR, the position behind the last token standing for no predecessor; lists short
and long (held by groups of lanes up to 512 tokens, beyond that fetched at every look, and beyond 63 predecessors from the bitmap)."""
import numpy as np
import pytest
import torch

import paper_2504_08966_amd as P
from oracle import pact_oracle as O
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


# whole words of the bitmap and one more; one and two turns of the second look
@pytest.mark.parametrize("n", [1088, 1089, 2048, 2049, 4096, 4161])
@pytest.mark.parametrize("blob,d_c", [(4, 0.02), (12, 0.02), (40, 0.02), (90, 0.03)])      # neighbours of a token: a few, dozens, more than a record holds
def test_centres_and_assignment(n, blob, d_c):
    r = np.random.default_rng(n + blob)
    dk = 64
    cen = r.normal(size=(n // blob + 1, dk))
    u = cen[r.integers(0, len(cen), n)] / np.sqrt(dk) + 0.14 * r.normal(size=(n, dk)) / np.sqrt(dk)
    u = u.astype(np.float32)
    o = P.dbdpc_cluster(gu.dev(u, "f32"), d_c, 2.0)
    torch.cuda.synchronize()
    rep = P.read_report(o["rep"])
    ref = O.dbdpc(u.astype(np.float64), d_c, 2.0)
    assert rep["n_centers"] == ref["centers"].size and rep["refine_overflow"] == 0
    assert np.array_equal(o["center_idx"][:rep["n_centers"]].cpu().numpy(), ref["centers"])
    assert np.array_equal(o["cluster_id"].cpu().numpy(), ref["labels"])
