"""The density order behind the centre selection (Alg. 2): the densities that decide it, what happens where
the fp32-term sums had it wrong, and that a call's densities are the same on every run."""
import numpy as np
import pytest
import torch

import paper_2504_08966_amd as P
from oracle import pact_oracle as po

pytestmark = pytest.mark.gpu
LOG2E = 1.4426950408889634


def _alike_with_copies(n, triples, d_n, seed):
    """64-wide bf16 keys that are nearly all alike, and among them `triples` times three parallel keys v c, 2 v c and v c', whose true
    densities are equal: the density pass's factor of the first two, 1/|v c| sqrt(log2(e) / d_n) in fp32, is rounded up by more than
    the band stands for (all terms of a token share it), that of the third hardly.  (v holds integers up to 15 and c is at most 17, so
    that the products are bf16 numbers.)"""
    r = np.random.default_rng(seed)
    base = r.standard_normal(64)
    base *= 10.0 / np.abs(base).max()
    v = np.clip(np.rint(base + r.standard_normal((n, 64))), -15, 15)
    scales = np.arange(1, 18, 2, dtype=np.float64)
    a = np.float32(LOG2E) / np.float32(d_n)
    inv = 1.0 / (np.linalg.norm(v, axis=1)[:, None] * scales)
    err = (inv.astype(np.float32) * np.sqrt(a)).astype(np.float64) / (inv * np.sqrt(np.float64(a))) - 1.0
    u = v[:400] / np.linalg.norm(v[:400], axis=1)[:, None]
    term = np.exp(-(1.0 - np.mean(u @ u.T)) / d_n)                       # of a typical pair
    band = 2.0 ** -20 * (1.0 + 4.0 * LOG2E / d_n) * np.sqrt(n * term)
    need = band / (0.9 * n * term / d_n)
    level = np.where((err > 1e-9) & (err < 1e-8), scales, 0.0).max(axis=1)
    pick = np.flatnonzero((err.max(axis=1) > need + 1.2e-8) & (level > 0))[:triples]
    assert pick.size == triples
    up = scales[np.argmax(err, axis=1)][pick, None]
    x = v * r.choice(scales, n)[:, None]
    x[pick] = v[pick] * up
    twin, third = np.setdiff1d(np.arange(n), pick)[:2 * triples].reshape(2, triples)
    x[twin], x[third] = 2.0 * v[pick] * up, v[pick] * level[pick, None]
    at = r.permutation(n)                                                # token i goes to row at[i]
    out = np.empty((n, 64), dtype=np.float32)
    out[at] = x
    return out, at[np.stack([pick, twin, third])]


def _distances(x):
    """Eq. 5 in fp64 (plain torch, on the GPU)."""
    u = x.double()
    u = u / u.norm(dim=1, keepdim=True)
    d = (1.0 - u @ u.T).clamp_(0.0, 2.0)
    d.fill_diagonal_(0.0)
    return d


def _centres_of(near, rho):
    """Alg. 2's loop on given densities (equal ones by index)."""
    blocked, centres = np.zeros(rho.size, dtype=bool), []
    for i in po.density_order(rho):
        if not blocked[i]:
            centres.append(int(i))
            blocked |= near[i]
    return np.array(sorted(centres))


@pytest.mark.parametrize("n,d_n", [(8000, 0.3), (8000, 0.4)])
def test_tokens_that_move_past_the_band_leave_one_order(n, d_n):
    # Of three parallel keys two are evaluated again, since their sums are equal, and the third is not: its sum is further away than the
    # band.  The two fp64 densities then fall behind the third one: its list of predecessors, which names them, has to be
    # made again with theirs, which name it (otherwise the three wait for each other for good).
    keys, role = _alike_with_copies(n, 100, d_n, 3)
    x = torch.from_numpy(keys).cuda().to(torch.bfloat16)
    d_c = 1e-6                                                  # parallel keys are the only neighbours
    # the fp32-term sums: with one of the three there are no neighbours, hence nothing is evaluated again; each of the other two adds 1
    sums = np.zeros(n)
    for k in range(3):
        idx = np.setdiff1d(np.arange(n), np.delete(role, k, axis=0))
        o = P.dbdpc_cluster(x, d_c, d_n, idx=torch.from_numpy(idx).int().cuda(),
                            n_idx_dev=torch.tensor([idx.size], dtype=torch.int32, device="cuda"), want_rho=True)
        rep = P.read_report(o["rep"])
        assert rep["rho_rechecked"] == 0 and rep["refine_overflow"] == 0, rep
        sums[idx] = o["rho"].cpu().numpy()[:idx.size] + 2.0
    o = P.dbdpc_cluster(x, d_c, d_n, want_rho=True, want_rank=True)
    torch.cuda.synchronize()
    rep, rho, rank = P.read_report(o["rep"]), o["rho"].cpu().numpy(), o["rank"].cpu().numpy()
    first, third = role[0], role[2]
    passed = (sums[first] > sums[third]) & (rho[first] < rho[third])
    print(f"n={n} d_n={d_n}: listed {rep['rho_rechecked']}, passed {passed.sum()}, centres {rep['n_centers']}")
    assert rep["rho_rechecked"] >= 200 and rep["refine_overflow"] == 0 and passed.sum() >= 20
    d = _distances(x)
    exact = torch.exp(-d / float(np.float32(d_n))).sum(1).cpu().numpy()
    assert np.max(np.abs(rho[first] - exact[first])) <= 1e-10 * exact.max()          # those are the fp64 values
    order = np.empty(n, dtype=np.int64)
    order[rank] = np.arange(n)
    assert np.array_equal(order, po.density_order(rho))
    assert np.array_equal(o["center_idx"][:rep["n_centers"]].cpu().numpy(), _centres_of((d <= d_c).cpu().numpy(), rho))


@pytest.mark.parametrize("n,dk,dtype,d_n", [(1500, 512, torch.bfloat16, 0.05), (4500, 128, torch.bfloat16, 0.02), (2700, 64, torch.float32, 0.1),
                                            (2048, 1024, torch.bfloat16, 0.2), (2048, 1024, torch.bfloat16, 0.21)])
def test_densities_do_not_depend_on_the_order_of_the_additions(n, dk, dtype, d_n):
    # Below d_n = 0.21 the terms span more binades than an fp64 sum holds: wavefronts add their parts in whatever order they get there.
    r = np.random.default_rng(n)
    x = r.standard_normal((12, dk))[r.integers(0, 12, n)] * 3.0 + r.standard_normal((n, dk))
    x = torch.from_numpy(x.astype(np.float32)).cuda().to(dtype)
    ws = P.alloc_workspace(n, 1, dk, 1, 1, key_dtype=dtype)
    runs = [P.dbdpc_cluster(x, 0.0, d_n, ws=ws, want_rho=True)["rho"] for _ in range(12)]
    for k in runs[1:]:
        assert torch.equal(k, runs[0]), f"{int((k != runs[0]).sum())} densities differ between two runs"
    # and they are the sums: a term's error is that of its exponent, (dk + 16) 2^-24 / d_n at the very most and mostly far less
    exact = torch.exp(-_distances(x) / float(np.float32(d_n))).sum(1)
    assert float(((runs[0] - exact).abs() / exact).max()) <= (dk + 16) * 2.0 ** -24 / d_n


def _twins(n, dk, spread, seed):
    """fp32 keys of which the last half of the tokens `spread` names are the first half again, off by one part in 10^6: densities that differ
    by less than the fp32 terms can tell."""
    r = np.random.default_rng(seed)
    first, second = spread
    x = r.standard_normal((max(2, n // 12), dk))[r.integers(0, max(2, n // 12), n)] + 0.25 * r.standard_normal((n, dk))
    x[second] = x[first] + 1e-6 * r.standard_normal((len(first), dk))
    return x.astype(np.float32)


def _order_of_sums(x, d_n, idx=None):
    """Densities as the fp32 terms leave them (no neighbours within 0: nothing is evaluated again) and in fp64."""
    n = x.shape[0]
    kw = {} if idx is None else dict(idx=torch.from_numpy(idx).int().cuda(), n_idx_dev=torch.tensor([idx.size], dtype=torch.int32, device="cuda"))
    o = P.dbdpc_cluster(x, 0.0, d_n, want_rho=True, **kw)
    rep = P.read_report(o["rep"])
    assert rep["rho_rechecked"] == 0 and rep["refine_overflow"] == 0, rep
    u = x if idx is None else x[torch.from_numpy(idx).cuda()]
    d = _distances(u)
    return o["rho"].cpu().numpy()[:n if idx is None else idx.size], torch.exp(-d / float(np.float32(d_n))).sum(1).cpu().numpy(), d


def _check_reordered(x, d_c, d_n, idx, sums, exact, d, first, second):
    """The call's centres are those of the fp64 order, which the fp32-term sums get wrong for some pairs (first[k], second[k])."""
    kw = {} if idx is None else dict(idx=torch.from_numpy(idx).int().cuda(), n_idx_dev=torch.tensor([idx.size], dtype=torch.int32, device="cuda"))
    wrong = np.sign(sums[first] - sums[second]) != np.sign(exact[first] - exact[second])
    near = (d <= float(np.float32(d_c))).cpu().numpy()
    assert wrong.sum() >= 1 and near[first, second].all()
    for _ in range(3):
        o = P.dbdpc_cluster(x, d_c, d_n, want_rho=True, **kw)
        torch.cuda.synchronize()
        rep, rho = P.read_report(o["rep"]), o["rho"].cpu().numpy()[:exact.size]
        assert rep["rho_rechecked"] >= 2 and rep["refine_overflow"] == 0
        assert np.max(np.abs(rho[first] - exact[first])) <= 1e-11 * exact.max()
        centres = _centres_of(near, rho)
        tokens = centres if idx is None else idx[centres]
        assert np.array_equal(o["center_idx"][:rep["n_centers"]].cpu().numpy(), tokens)
        assert not np.array_equal(centres, _centres_of(near, sums))           # (the selection before the re-evaluation had others)
    print(f"{wrong.sum()} of {first.size} pairs in the wrong order, listed {rep['rho_rechecked']}, rounds {rep['rounds']}")


@pytest.mark.parametrize("n,pairs,dk", [(960, 480, 4096), (1000, 300, 512)])
def test_selection_runs_again_when_the_fp64_densities_are_the_last_to_come(n, pairs, dk):
    # hundreds of listed tokens with long rows: the re-evaluation ends long after the selection, whose order it changes
    # (a build that noted which workgroup ran it again: one of the re-evaluation's, in all calls)
    first, second = np.arange(pairs), np.arange(n - pairs, n)
    x = torch.from_numpy(_twins(n, dk, (first, second), n)).cuda()
    sums, exact, d = _order_of_sums(x, 2.0)
    _check_reordered(x, 1e-5, 2.0, None, sums, exact, d, first, second)


def test_selection_runs_again_when_it_is_the_last_to_come():
    # Two listed tokens, and a selection that has to go along a chain: tokens on an arc, densest at one end. Of the twins one pair whose order the
    # fp32-term sums get wrong is left in.  (The same build: the selection's own workgroup.)
    n, arc, dk, d_c = 2620, 2000, 64, 2e-3
    r = np.random.default_rng(5)
    first, second = np.arange(n - 120, n - 60), np.arange(n - 60, n)
    x = _twins(n, dk, (first, second), 5)
    x[first] = r.standard_normal((60, dk))                                    # (no neighbours but their twins)
    x[second] = x[first] + 1e-6 * r.standard_normal((60, dk))
    theta = np.concatenate([np.linspace(0.0, 2.5, arc), 0.4 * r.random(n - 120 - arc)])
    x[:n - 120] = 1e-4 * r.standard_normal((n - 120, dk))
    x[:n - 120, 0] += np.cos(theta)
    x[:n - 120, 1] += np.sin(theta)
    x = torch.from_numpy(x.astype(np.float32)).cuda()
    for k in range(60):
        idx = np.concatenate([np.arange(n - 60), second[k:k + 1]])
        sums, exact, d = _order_of_sums(x, 2.0, idx)
        a, b = n - 120 + k, n - 60                                            # their positions in the subset
        if np.sign(sums[a] - sums[b]) != np.sign(exact[a] - exact[b]):
            return _check_reordered(x, d_c, 2.0, idx, sums, exact, d, np.array([a]), np.array([b]))
    pytest.fail("no pair whose order the sums get wrong")
