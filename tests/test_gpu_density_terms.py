"""Density sums: terms between two powers of two are summed as integers, others in fp64, whatever the cutoff's scale and the rows' angles;
the list of undecided pairs in parts."""
import numpy as np
import pytest
import torch

import paper_2504_08966_amd as P
from oracle import pact_oracle as po
from tests import gpu_util as gu
from tests.test_gpu_parity import _mk, assert_same, oracle_reduce

pytestmark = pytest.mark.gpu


# d_n: of unrelated rows one power of two, the next, none; sums in two parts.  Angles: unrelated rows, all in a cone (all terms near 1), some
# opposite (blocks of both kinds beside each other), rows that are copies.  Sizes: a part of a tile, whole tiles, one token more, mirrored ones
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d_n", [5.0, 2.0, 1.0, 0.5, 0.3, 0.2])
@pytest.mark.parametrize("n,dk,angles", [(61, 64, "any"), (128, 64, "opposite"), (1025, 64, "opposite"), (1025, 128, "cone"), (2433, 64, "any"), (3970, 128, "opposite")])
def test_densities(n, dk, angles, d_n, dtype):
    rng = np.random.default_rng(8000 + n)
    U = rng.normal(size=(n, dk))
    if angles == "cone":
        U[:, 0] += 40.0
    if angles == "opposite":
        U[n // 3: n // 3 + 70] = -U[:70] + 0.05 * rng.normal(size=(min(70, n - n // 3), dk))
    U[5] = U[40]
    U = gu.dev(U, dtype).float().cpu().numpy().astype(np.float64)
    out = P.dbdpc_cluster(gu.dev(U, dtype), 1e-4, d_n, want_rho=True)
    torch.cuda.synchronize()
    got = out["rho"].cpu().numpy()
    ref = po.dbdpc(U, float(np.float32(1e-4)), float(np.float32(d_n)))
    # relative error of a term: its distance's, at worst (dk + 16) 2^-23 and a quarter of that as it is met, over d_n; its exponent's rounding; v_exp_f32's 2^-23
    np.testing.assert_allclose(got, ref["rho"], rtol=(dk + 16) * 2.0 ** -25 / d_n + 2.0 ** -23 * (2.0 + 2.0 / d_n), atol=0)
    assert got[5] == got[40]
    rep = P.read_report(out["rep"])
    assert np.array_equal(out["center_idx"][: rep["n_centers"]].cpu().numpy(), ref["centers"])


@pytest.mark.parametrize("n,half", [(1025, 70), (1025, 95), (1300, 100), (2600, 128)])
def test_undecided_pairs_of_few_workgroups(n, half):
    # two blocks of identical keys at a distance of d_c to within fp32 rounding: of one tile come more pairs than a part of the list holds (8192)
    k = np.zeros((n, 1, 16), dtype=np.float32)
    k[:half, 0, 0] = 1.0
    k[half:2 * half, 0, 0] = 0.9
    k[half:2 * half, 0, 1] = np.float32(np.sqrt(1.0 - 0.81))
    k[2 * half:, 0, 2:] = np.random.default_rng(13).normal(size=(n - 2 * half, 14)).astype(np.float32)
    a, b = k[0, 0].astype(np.float64), k[half, 0].astype(np.float64)
    at = 1.0 - a @ b / np.sqrt((a @ a) * (b @ b))
    s = _mk(k)
    for d_c in (np.nextafter(np.float32(at), np.float32(0)), np.nextafter(np.float32(at), np.float32(1))):
        g = gu.gpu_reduce(s, float(d_c), lam=0.0)
        assert g["rep"]["refine_overflow"] == 0 and 2 * half * half <= g["rep"]["dc_checked_pairs"] < 65536
        assert_same(g, oracle_reduce(s, float(d_c), lam=0.0), s, f"n={n} d_c={d_c}")


def _two_blocks(n, half):
    """Two blocks of identical keys ahead of other rows, and the distance of the two."""
    k = np.zeros((n, 1, 16), dtype=np.float32)
    k[:half, 0, 0] = 1.0
    k[half:2 * half, 0, 0] = 0.9
    k[half:2 * half, 0, 1] = np.float32(np.sqrt(1.0 - 0.81))
    k[2 * half:, 0, 2:] = np.random.default_rng(14).normal(size=(n - 2 * half, 14)).astype(np.float32)
    a, b = k[0, 0].astype(np.float64), k[half, 0].astype(np.float64)
    return _mk(k), float(np.float32(1.0 - a @ b / np.sqrt((a @ a) * (b @ b))))


# a list in parts that is nearly full (every ordered pair takes a place of 65536: tiles on both sides of the diagonal), one place after another of all parts
@pytest.mark.parametrize("n", [1025, 1100, 1300])
def test_a_nearly_full_list_of_undecided_pairs(n):
    s, d_c = _two_blocks(n, 180)
    g = gu.gpu_reduce(s, d_c, lam=0.0)
    assert g["rep"]["refine_overflow"] == 0 and g["rep"]["dc_checked_pairs"] == 2 * 180 * 180
    assert_same(g, oracle_reduce(s, d_c, lam=0.0), s, f"n={n}")


# more pairs than all parts hold, by a few and by far (mirrored tiles and others), alone and in a batch beside a sample that has none: said of the one, and its outputs are well-formed
@pytest.mark.parametrize("n,half", [(1100, 260), (1300, 600), (2600, 400), (4100, 1000), (4100, 2000)])
@pytest.mark.parametrize("batch", [1, 2, 3])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_more_undecided_pairs_than_a_list_holds(n, half, batch, dtype):
    s, _ = _two_blocks(n, half)
    keys, hid, q = gu.dev(s.keys.reshape(n, -1), dtype), gu.dev(s.hidden, dtype), gu.dev(s.queries.reshape(n, -1), dtype)
    a, b = keys[0].double(), keys[half].double()
    d_c = float(np.float32((1.0 - (a @ b) / torch.sqrt((a @ a) * (b @ b))).item()))
    many = batch - 1 if batch > 1 else 1                                       # samples that are this one; the last of a batch is its last 1030 rows' worth of others
    other = torch.randn(1030, 16, device="cuda", generator=torch.Generator("cuda").manual_seed(3)).to(keys.dtype)
    lens = [n] * many + [1030] * (batch - many)
    ks = torch.cat([keys] * many + [other] * (batch - many))
    hs = torch.cat([hid] * many + [hid[:1030]] * (batch - many))
    qs = torch.cat([q] * many + [q[:1030]] * (batch - many))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(int)
    for _ in range(2):                                                         # (the second finds the counters as the first left them)
        o = P.pact_reduce_varlen(hs, ks, ks, qs, 1, 16, 1, off.tolist(), [P.PactParams(0.0, d_c, 2.0, 1.5)] * batch)
        torch.cuda.synchronize()
        for k in range(batch):
            g = gu.trim(o, lens[k], int(off[k]), k)
            rep, C = g["rep"], g["rep"]["n_centers"]
            assert rep["n_kept"] == lens[k]
            if k < many:
                assert rep["refine_overflow"] & 1 and rep["dc_checked_pairs"] == 65536
            else:
                assert rep["refine_overflow"] == 0 and rep["dc_checked_pairs"] < 65536
            assert g["cluster_id"].min() >= 0 and g["cluster_id"].max() == C - 1
            assert g["counts"].sum() == lens[k] and np.array_equal(np.bincount(g["cluster_id"], minlength=C), g["counts"])


# Sums of float bits and of fp64 terms are the same only if no term of an exponent at or above -k is below 2^-k, and none at or below it above.  Two kinds of rows, all pairs of unlike ones
# with the same exponent (an axis of its own keeps each row away from its like), which moves over -k by its last places with d_n: kinds in blocks of 128 (summed as bits), and mixed, with a row
# of a third kind in every 64 (fp64)
@pytest.mark.parametrize("k", range(1, 13))
def test_terms_at_powers_of_two(k):
    n, c, own = 256, -0.9, 0.25
    kind = np.arange(n) // 128
    rows = np.zeros((n + 4, n + 4))
    rows[:n, 0] = np.where(kind, c, 1.0)
    rows[:n, 1] = np.where(kind, np.sqrt(1 - c * c), 0.0)
    rows[np.arange(n), 2 + np.arange(n)] = own
    rows[n:, n + 2] = 1.0
    rows[n:, n + 3] = [0.3, 0.6, 0.9, 1.2]
    perm = np.random.default_rng(k).permutation(n)
    mixed = np.insert(perm, [0, 64, 128, 192], np.arange(n, n + 4))
    assert len(set(mixed)) == n + 4
    keys = gu.dev(rows, "f32")
    other = keys[torch.from_numpy(mixed).cuda()].contiguous()
    d_n = np.float32(1.4426950408889634 * (1.0 - c / (1.0 + own * own)) / k)   # exponent of unlike rows: -k
    assert d_n >= 0.21                                                         # (below, sums are in two parts)
    seen = set()
    for _ in range(12):
        d_n = np.nextafter(d_n, np.float32(0))
    for _ in range(25):
        a = P.dbdpc_cluster(keys, 1e-4, float(d_n), want_rho=True)
        b = P.dbdpc_cluster(other, 1e-4, float(d_n), want_rho=True)
        torch.cuda.synchronize()
        assert P.read_report(a["rep"])["rho_rechecked"] == 0                   # (the sums themselves)
        ra, rb = a["rho"].cpu().numpy(), b["rho"].cpu().numpy()
        assert np.array_equal(ra[mixed], rb), (k, d_n)
        seen.add(ra[0])
        d_n = np.nextafter(d_n, np.float32(10))
    assert len(seen) > 4                                                       # (the terms did move)
