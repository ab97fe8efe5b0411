"""Clustering rows of more than 2 KB: undecided pairs by an fp32 screen first, the assignment of bf16 rows by 16 x 16 products.  Against the oracle."""
import numpy as np
import pytest
import torch

import paper_2504_08966_amd as P
from oracle import pact_oracle as O
from pact_synth import gen
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _check(u, dtype, d_c, d_n=2.0):
    o = P.dbdpc_cluster(gu.dev(u, dtype), d_c, d_n)
    torch.cuda.synchronize()
    rep = P.read_report(o["rep"])
    ref = O.dbdpc(u.astype(np.float64), float(np.float32(d_c)), float(np.float32(d_n)))
    assert rep["n_centers"] == ref["centers"].size and not rep["refine_overflow"] & 1          # (bit 1: many tokens with equal densities)
    assert np.array_equal(o["center_idx"][:rep["n_centers"]].cpu().numpy(), ref["centers"])
    assert np.array_equal(o["cluster_id"].cpu().numpy(), ref["labels"])
    return rep, ref


# bf16 rows below 3.5 KB take the products from 6 MB of them on (the last size; the first three are compared by wavefronts);
# widths of whole and broken 64-byte steps and wavefronts' parts; a last sixteen of one token; one, two and more turns of 32 centres in reach
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,dk,blob", [(2, 1032, 1), (17, 1032, 6), (300, 1544, 24), (1009, 2048, 24), (700, 3584, 100), (1201, 4104, 40),
                                       (2, 1800, 1), (17, 1800, 6), (300, 2056, 24), (3001, 1032, 24)])
def test_neighbours_near_the_cutoff(n, dk, blob, dtype):
    r = np.random.default_rng(n + dk)
    cen = r.normal(size=(n // blob + 1, dk))
    u = cen[np.arange(n) // blob] / np.sqrt(dk) + 0.148 * r.normal(size=(n, dk)) / np.sqrt(dk)     # distances within a blob about 0.0215
    u = (gen.round_to_bf16(u) if dtype == "bf16" else u).astype(np.float32)
    rep, ref = _check(u, dtype, 0.0215)
    if n > 100:
        assert rep["dc_checked_pairs"] > 50 and n // 8 < rep["n_centers"] < n


# Tokens at exactly one distance of many centres (sums of unit vectors, each of which stands there twice and is denser): more than are kept per token, then
# more in a group of 16 tokens than its list holds.  The lowest index is the nearest.
@pytest.mark.parametrize("spread,hubs", [(6, 20), (9, 20), (12, 33), (80, 16)])
def test_many_centres_at_one_distance(spread, hubs):
    dk, units = 2048, 1300
    r = np.random.default_rng(spread)
    e = np.zeros((units, dk), np.float32)
    e[np.arange(units), r.permutation(dk)[:units]] = 1.0
    hub = np.stack([e[(np.arange(spread) + k * spread) % units if spread * hubs <= units else (np.arange(spread) + k * 81) % units].sum(0) for k in range(hubs)])
    u = np.concatenate([e[:700], hub, e[700:], e])          # (hubs in the middle of the sequence)
    d_c = 1.0 - 0.9 / np.sqrt(spread)
    rep, ref = _check(u, "bf16", d_c, 0.15)                # (a normaliser with which the hubs are the less dense)
    assert rep["n_centers"] == units
