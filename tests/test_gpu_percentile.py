"""The percentile split on given scores, at the edges of what a workgroup's wavefronts and registers hold, against the same selection in
numpy on the order that the fp32 bit patterns have."""
import numpy as np
import pytest
import torch

import paper_2504_08966_amd as P

pytestmark = pytest.mark.gpu


def _keys(f):
    u = f.view(np.uint32)
    return np.where(u >> 31 != 0, ~u, u | np.uint32(0x80000000))


def _scores(kind, n, r):
    f = np.exp(0.5 * r.standard_normal(n)).astype(np.float32)
    if kind == "ties":                                # more of them in a bin than one wavefront ranks
        f = r.integers(1, 4, n).astype(np.float32)
    elif kind == "near":                              # neighbours in the last place
        f = (np.float32(1.0).view(np.uint32) + r.integers(0, 60, n).astype(np.uint32)).view(np.float32)
    elif kind == "odd":
        f *= np.where(r.random(n) < 0.3, -1.0, 1.0).astype(np.float32)
        f[r.random(n) < 0.1] = np.nan
        f[r.random(n) < 0.05] = np.inf
        f[r.random(n) < 0.05] = -np.inf
        f[r.random(n) < 0.05] = 0.0
    return f


@pytest.mark.parametrize("kind", ["smooth", "ties", "near", "odd"])
@pytest.mark.parametrize("n", [1, 2, 63, 65, 1000, 1024, 1025, 4095, 4096, 4097, 8192, 8193, 16384, 16385, 20001, 32768])
def test_split(n, kind):
    r = np.random.default_rng(n)
    for lam in (0.0, 0.3, 0.45, 0.999, 1.0):
        f = _scores(kind, n, r)
        kept, pruned, rep = P.pact_prune(torch.from_numpy(f).cuda(), lam)
        torch.cuda.synchronize()
        rep = P.read_report(rep)
        key = _keys(f)
        m = min(int(np.floor(np.float64(np.float32(lam)) * n)), n - 1)
        at = np.argsort(key, kind="stable")[m]
        keep = key >= key[at]
        assert np.array_equal(kept[: rep["n_kept"]].cpu().numpy(), np.flatnonzero(keep))
        assert np.array_equal(pruned[: rep["n_pruned"]].cpu().numpy(), np.flatnonzero(~keep))
        tau, d = np.float64(f[at]), f.astype(np.float64)
        with np.errstate(invalid="ignore"):
            near = (key != key[at]) & (np.abs(d - tau) <= 1e-6 * np.abs(tau))
        assert rep["score_near_ties"] == near.sum() and rep["nonfinite_seen"] == (~np.isfinite(f)).sum()
