"""Candidate pass of fp32 keys by the upper two bytes of each element (more than one turn of 128 x 64 tiles) and by three: clusters and recovery
against the oracle, with rows whose margin is the ordinary one, and with rows that are mostly one element."""
import numpy as np
import pytest
import torch

import paper_2504_08966_amd as P
from oracle import pact_oracle as O
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _keys(kind, n, dk, r):
    nb = max(2, n // 12)
    k = r.normal(size=(nb, dk))[r.integers(0, nb, n)] + 0.17 * r.normal(size=(n, dk))
    if kind != "flat":                                     # one element that is most of the row: in a few rows, in all
        rows = np.arange(0, n, 97) if kind == "some" else np.arange(n)
        k[rows, rows % 3 if kind == "some" else 0] += (40.0 if kind == "some" else 12.0) * np.sqrt(dk) / 8.0
    return (k * np.exp(r.normal(0, 0.5, (n, 1)))).astype(np.float32)


# three bytes in halves and in whole tiles, two bytes (the last two sizes); one and several slices; recovery that reaches some tokens and not others
@pytest.mark.parametrize("kind", ["flat", "some", "all"])
@pytest.mark.parametrize("n,n_kv,d_h", [(1100, 1, 64), (2500, 1, 200), (5000, 4, 128), (6100, 1, 64), (6250, 2, 100)])
def test_recovery(n, n_kv, d_h, kind):
    r = np.random.default_rng(n + d_h)
    dk, lam, h = n_kv * d_h, 0.5, 64
    keys = _keys(kind, n, dk, r)
    hid, q = r.normal(size=(n, h)).astype(np.float32), r.normal(size=(n, dk)).astype(np.float32) / np.sqrt(d_h).astype(np.float32)
    d_c = {"flat": 0.022, "some": 0.02, "all": 0.012}[kind]
    ref = O.pact_reduce(hid, keys.reshape(n, n_kv, d_h), q.reshape(n, n_kv, d_h), keys.reshape(n, n_kv, d_h), lam, float(np.float32(d_c)), 2.0, 1.5)
    k = gu.dev(keys, "f32")
    o = P.pact_reduce(gu.dev(hid, "f32"), k, k, gu.dev(q, "f32"), n_kv, d_h, n_kv, P.PactParams(lam, d_c, 2.0, 1.5))
    torch.cuda.synchronize()
    rep = P.read_report(o["rep"])
    assert 0 < rep["n_reincorporated"] and rep["score_near_ties"] == 0
    assert np.array_equal(o["cluster_id"].cpu().numpy(), ref["cluster_id"])
