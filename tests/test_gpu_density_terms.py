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


@pytest.mark.parametrize("n,half", [(1025, 70), (1300, 100), (2600, 128)])
def test_undecided_pairs_of_few_workgroups(n, half):
    # two blocks of identical keys at a distance of d_c to within fp32 rounding: of one tile come more pairs than a part of the list holds (4096)
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
