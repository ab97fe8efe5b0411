"""Precision of the matrix passes on fp32 keys: single cosines against 64 bits, over rows whose largest element is anything from
one among equals to all there is."""
import numpy as np
import pytest
import torch

import paper_2504_08966_amd as P

pytestmark = pytest.mark.gpu


def _rows(kind, n, dk, r):
    x = r.standard_normal((n, dk))
    at = r.integers(0, dk, n) if kind != "channel" else np.full(n, dk // 3)
    if kind != "gauss":                            # one element of `kind` times the others' rms (a channel: of 8 times, in the same place)
        sign = 1.0 if kind == "channel" else np.where(r.random(n) < 0.5, -1.0, 1.0)
        x[np.arange(n), at] = (8.0 if kind == "channel" else float(kind)) * sign
    return (x * np.exp(0.5 * r.standard_normal((n, 1)))).astype(np.float32)


@pytest.mark.parametrize("dk", [128, 512, 3584])
@pytest.mark.parametrize("kind", ["gauss", "7.9", "channel", "12", "64", "65536"])
def test_cosines_of_fp32_keys(kind, dk):
    # The density of one of two tokens is 1 + exp(-d / d_n): with d_n = 0.05 it tells d to 1e-8.  An exponent d log2(e) / d_n of
    # up to 35 is rounded to 2^-19 (half an ulp) at most, which is 6.6e-8 of a cosine, 3.8e-8 rms; a term to 2^-23 d_n = 6e-9; the
    # scaling factors are within 2^-23 of the cosine; and 1.2e-8 rms is what the passes may leave out.
    d_n, n = 0.05, 240
    r = np.random.default_rng(dk)
    x = _rows(kind, n, dk, r)
    u = x.astype(np.float64) / np.linalg.norm(x.astype(np.float64), axis=1, keepdims=True)
    cos = (u[0::2] * u[1::2]).sum(1)
    t = np.exp(-(1.0 - cos) / np.float64(np.float32(d_n)))
    keys = torch.from_numpy(x).cuda()
    ws = P.alloc_workspace(2, 1, dk, 1, 1, key_dtype=torch.float32)
    rho = torch.stack([P.dbdpc_cluster(keys[i:i + 2], 0.0, d_n, ws=ws, want_rho=True)["rho"] for i in range(0, n, 2)]).cpu().numpy()
    assert np.array_equal(rho[:, 0], rho[:, 1])
    ok = t > 1e-10                                  # (1 + t is rounded to 2^-53)
    err = (np.log((rho[ok, 0] - 1.0) / t[ok]) * d_n)
    rms, scale = np.sqrt(np.mean(err ** 2)), np.sqrt(np.mean((cos[ok] * 2.0 ** -23) ** 2))
    print(f"{kind} {dk}: {ok.sum()} pairs, rms {rms:.2e}, largest {np.abs(err).max():.2e}")
    assert ok.sum() >= 60 and rms <= np.sqrt(3.8e-8 ** 2 + 6e-9 ** 2 + 1.2e-8 ** 2 + scale ** 2)
