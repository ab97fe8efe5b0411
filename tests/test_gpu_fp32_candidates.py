"""Candidate pass of fp32 keys, in halves of its tiles and whole ones, one turn of the chip and several: clusters and recovery against the oracle, with
ordinary rows and with rows that are mostly one element."""
import numpy as np
import pytest
import torch

import paper_2504_08966_amd as P
from oracle import pact_oracle as O
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _keys(kind, n, dk, r, per=12):
    nb = max(2, n // per)
    k = r.normal(size=(nb, dk))[r.integers(0, nb, n)] + 0.17 * r.normal(size=(n, dk))
    if kind != "flat":                                     # one element that is most of the row: in a few rows, in all
        rows = np.arange(0, n, 97) if kind == "some" else np.arange(n)
        k[rows, rows % 3 if kind == "some" else 0] += (40.0 if kind == "some" else 12.0) * np.sqrt(dk) / 8.0
    return (k * np.exp(r.normal(0, 0.5, (n, 1)))).astype(np.float32)


# halves and whole tiles, one turn and more; one and several slices; recovery that reaches some tokens and not others
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


# more than 64 groups of 64 centres: the loops over further groups
@pytest.mark.parametrize("kind", ["flat", "all"])
def test_recovery_among_more_than_4096_centres(kind):
    n, dk, lam, d_c = 12000, 64, 0.45, {"flat": 0.022, "all": 0.0055}[kind]
    r = np.random.default_rng(5)
    keys = _keys(kind, n, dk, r, per=1)
    hid, q = r.normal(size=(n, 16)).astype(np.float32), r.normal(size=(n, dk)).astype(np.float32) / 8
    one = lambda x: x.reshape(n, 1, dk)
    ref = O.pact_reduce(hid, one(keys), one(q), one(keys), lam, float(np.float32(d_c)), 2.0, 1.5)
    k = gu.dev(keys, "f32")
    o = P.pact_reduce(gu.dev(hid, "f32"), k, k, gu.dev(q, "f32"), 1, dk, 1, P.PactParams(lam, d_c, 2.0, 1.5))
    torch.cuda.synchronize()
    rep = P.read_report(o["rep"])
    assert rep["n_centers"] > 4096 + 64 and rep["n_reincorporated"] > 500 and rep["score_near_ties"] == 0
    assert np.array_equal(o["cluster_id"].cpu().numpy(), ref["cluster_id"])


# samples that start inside the batch, among them one of a few tokens and one of none pruned
@pytest.mark.parametrize("kind,d_c", [("flat", 0.022), ("some", 0.02), ("all", 0.012)])
@pytest.mark.parametrize("dk", [64, 200])
def test_recovery_in_batches(kind, d_c, dk):
    lens, lams = [4100, 5, 2500, 4001, 3, 3300], [0.5, 0.5, 0.6, 0.45, 0.0, 0.7]
    r = np.random.default_rng(dk)
    ks = [_keys(kind, n, dk, r) for n in lens]
    hs = [r.normal(size=(n, 16)).astype(np.float32) for n in lens]
    qs = [(r.normal(size=(n, dk)) / np.sqrt(dk)).astype(np.float32) for n in lens]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(int)
    k, h, q = (gu.dev(np.concatenate(x), "f32") for x in (ks, hs, qs))
    o = P.pact_reduce_varlen(h, k, k, q, 1, dk, 1, off.tolist(), [P.PactParams(lam, d_c, 2.0, 1.5) for lam in lams])
    torch.cuda.synchronize()
    reps = P.read_report(o["rep"])
    for b, n in enumerate(lens):
        one = lambda x: x.reshape(n, 1, dk)
        ref = O.pact_reduce(hs[b], one(ks[b]), one(qs[b]), one(ks[b]), lams[b], float(np.float32(d_c)), 2.0, 1.5)
        assert reps[b]["score_near_ties"] == 0 and (n < 2000 or reps[b]["n_reincorporated"] > n // 10), b
        assert np.array_equal(o["cluster_id"][off[b]:off[b + 1]].cpu().numpy(), ref["cluster_id"]), b
