"""What depends on the inputs alone: norms of several key rows per group of lanes (calls of enough rows, samples that start inside such a group), in each of the launches
that prepare keys; the query sums of long samples, which come in more chunks; hidden states' norms in two launches.  Against a call of one sample, whose rows are
taken one at a time, and the oracle."""
import numpy as np
import pytest
import torch

import paper_2504_08966_amd as P
from oracle import pact_oracle as O
from tests import gpu_util as gu
from tests.test_gpu_parity import _random_sample

pytestmark = pytest.mark.gpu


# 16, 32 and 64 lanes a row, one and two chunks a lane; batches with tokens enough for two, four or eight rows at a time, beside the splits as long as those are one turn of the chip (and the logits do not go head by head) and
# beside the logits, and with too few; a sample of its own never has enough
@pytest.mark.parametrize("dk,n_b,dtype", [(8, 165, "bf16"), (128, 165, "bf16"), (136, 165, "bf16"), (256, 165, "bf16"), (264, 100, "bf16"), (512, 100, "bf16"), (512, 400, "bf16"),
                                          (1024, 165, "bf16"), (4, 165, "f32"), (64, 165, "f32"), (68, 165, "f32"), (128, 165, "f32"), (132, 100, "f32"), (260, 165, "f32"), (512, 165, "f32"),
                                          (8, 850, "bf16"), (128, 850, "bf16"), (136, 440, "bf16"), (256, 880, "bf16"), (264, 230, "bf16"), (512, 600, "bf16"), (1024, 230, "bf16"), (1024, 500, "bf16"),
                                          (64, 500, "f32"), (68, 250, "f32"), (128, 450, "f32"), (512, 400, "f32")])
@pytest.mark.parametrize("d_n", [2.0, 0.1])
def test_several_rows_as_one_at_a_time(dk, n_b, dtype, d_n):
    lens = [n_b + k % 5 for k in range(31)] + [1, 2, 3]
    assert max(lens) <= 1024
    ss = [_random_sample(9100 + k, n, 1, 1, dk, 64, 0.3, dtype) for k, n in enumerate(lens)]
    hid, ks, qs = (gu.dev(np.concatenate([x(s).reshape(s.n, -1) for s in ss]), dtype) for x in (lambda s: s.hidden, lambda s: s.keys, lambda s: s.queries))
    ks[5] = 0                                              # a zero vector
    off = np.concatenate([[0], np.cumsum(lens)]).astype(int)
    prm = [P.PactParams(0.3, 0.06, d_n, 1.5) for _ in lens]
    o = P.pact_reduce_varlen(hid, ks, ks, qs, 1, dk, 1, off.tolist(), prm)
    torch.cuda.synchronize()
    reps = P.read_report(o["rep"])
    for k in range(len(lens)):
        a, b = off[k], off[k + 1]
        g = P.pact_reduce(hid[a:b], ks[a:b], ks[a:b], qs[a:b], 1, dk, 1, prm[k])
        torch.cuda.synchronize()
        rep = P.read_report(g["rep"])
        assert all(reps[k][f] == rep[f] for f in ("n_kept", "n_centers", "n_reincorporated", "zero_norm_seen")), k
        for name, m in (("scores", b - a), ("cluster_id", b - a), ("center_idx", rep["n_centers"]), ("merged", rep["n_centers"])):
            assert torch.equal(o[name][a:a + m], g[name][:m]), (k, name)


# one token more than eight chunks take, a last chunk of a few rows, and the widest queries that come in more chunks
@pytest.mark.parametrize("n,n_kv,n_q,d_h,dtype", [(8193, 1, 1, 64, "bf16"), (8193, 2, 2, 64, "f32"), (9217, 1, 8, 128, "bf16"), (12300, 1, 4, 32, "f32")])
def test_query_sums_of_long_samples(n, n_kv, n_q, d_h, dtype):
    s = _random_sample(31, n, n_kv, n_q, d_h, 64, 0.4, dtype)
    hid, ks, qs = (gu.dev(x.reshape(n, -1), dtype) for x in (s.hidden, s.keys, s.queries))
    got = P.pact_score(hid, ks, qs, n_kv, d_h, n_q)
    torch.cuda.synchronize()
    want = O.euti_scores(s.hidden, s.keys, s.queries)
    np.testing.assert_allclose(got[:n].cpu().numpy(), want, rtol=2e-7)          # one rounding to fp32: 6e-8, and the sums in fp64


# samples of one batch with 16, 10, 8, 6 and 1 chunks: each has its own number, that of a call of its own
@pytest.mark.parametrize("n_kv,n_q,d_h,dtype", [(1, 2, 32, "f32"), (2, 14, 64, "bf16"), (1, 3, 24, "f32")])
def test_query_sums_of_a_long_sample_beside_short_ones(n_kv, n_q, d_h, dtype):
    lens = [729, 17000, 100, 9500, 1024, 1]
    ss = [_random_sample(700 + k, n, n_kv, n_q, d_h, 64, 0.4, dtype) for k, n in enumerate(lens)]
    hid, ks, qs = (gu.dev(np.concatenate([x(s).reshape(s.n, -1) for s in ss]), dtype) for x in (lambda s: s.hidden, lambda s: s.keys, lambda s: s.queries))
    off = np.concatenate([[0], np.cumsum(lens)]).astype(int)
    o = P.pact_reduce_varlen(hid, ks, ks, qs, n_kv, d_h, n_q, off.tolist(), [P.PactParams(0.4, 0.02, 2.0, 1.5) for _ in lens])
    torch.cuda.synchronize()
    for k, s in enumerate(ss):
        a, b = off[k], off[k + 1]
        got = o["scores"][a:b]
        one = P.pact_score(hid[a:b], ks[a:b], qs[a:b], n_kv, d_h, n_q)
        torch.cuda.synchronize()
        assert torch.equal(got, one[:s.n]), k
        np.testing.assert_allclose(got.cpu().numpy(), O.euti_scores(s.hidden, s.keys, s.queries), rtol=2e-7)


# keys prepared beside the query sums (single samples of more than 4096 tokens with narrow queries), beside the split (with wide ones, or a query given as its mean) and beside the logits (shorter
# ones, batches); norms of the hidden states in the first launch, the second, part in either, with rows of one to four at a time
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("h,n_q,d_h", [(64, 1, 64), (1032, 1, 72), (3584, 2, 128), (256, 7, 64), (64, 9, 128)])
@pytest.mark.parametrize("mean", [False, True])
def test_inputs_in_any_launch(h, n_q, d_h, dtype, mean):
    lens = [1100, 4099, 17, 4097]
    rng = np.random.default_rng(77)
    hid, ks = (gu.dev(rng.normal(size=(sum(lens), c)), dtype) for c in (h, d_h))
    ks[1000:1040] = ks[0]
    qs = gu.dev(rng.normal(size=(len(lens) if mean else sum(lens), n_q * d_h)), dtype)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(int)
    prm = [P.PactParams(0.5, 0.1, 2.0, 1.5) for _ in lens]
    o = P.pact_reduce_varlen(hid, ks, ks, qs, 1, d_h, n_q, off.tolist(), prm)
    torch.cuda.synchronize()
    reps = P.read_report(o["rep"])
    norm = hid.double().cpu().norm(dim=1)
    for k in range(len(lens)):
        a, b = off[k], off[k + 1]
        q = qs[k:k + 1] if mean else qs[a:b]
        g = P.pact_reduce(hid[a:b], ks[a:b], ks[a:b], q, 1, d_h, n_q, prm[k])
        torch.cuda.synchronize()
        rep = P.read_report(g["rep"])
        assert all(reps[k][f] == rep[f] for f in ("n_kept", "n_centers", "n_reincorporated", "zero_norm_seen", "nonfinite_seen", "score_near_ties")), k
        for name, m in (("scores", b - a), ("cluster_id", b - a), ("center_idx", rep["n_centers"]), ("merged", rep["n_centers"]), ("cluster_counts", rep["n_centers"])):
            assert torch.equal(o[name][a:a + m], g[name][:m]), (k, name)
        # the scores in fp64, on the CPU
        Q = q.double().cpu().mean(0).reshape(n_q, d_h)
        want = norm[a:b] * torch.softmax(ks[a:b].double().cpu() @ Q.T, dim=0).mean(1)
        np.testing.assert_allclose(g["scores"][: b - a].cpu().numpy(), want.numpy(), rtol=2e-7)


# large batches, keys prepared beside the logits: their blocks evenly among those of the hidden states (one tensor as both keys) or ahead of them (two); one to four norms a wavefront, key blocks
# the more and the fewer; a query given as its mean leaves all norms to that launch
@pytest.mark.parametrize("h,n_q,d_h", [(64, 1, 64), (1032, 1, 8), (1032, 14, 64), (2560, 1, 128)])
@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("mean", [False, True])
def test_keys_among_hidden_states(h, n_q, d_h, two, mean):
    lens = [2500, 1, 4096, 1025, 3001, 2999] * 2 + [5900, 63]
    assert sum(lens) > 32768
    g = torch.Generator("cuda").manual_seed(11)
    rand = lambda *s: torch.randn(*s, device="cuda", generator=g).bfloat16()
    hid, ks, qs = rand(sum(lens), h), rand(sum(lens), d_h), rand(len(lens) if mean else sum(lens), n_q * d_h)
    ks[::7] = ks[3]
    pre = ks.clone() if two else ks
    off = np.concatenate([[0], np.cumsum(lens)]).astype(int)
    prm = [P.PactParams(0.5, 0.05, 2.0, 1.5) for _ in lens]
    o = P.pact_reduce_varlen(hid, pre, ks, qs, 1, d_h, n_q, off.tolist(), prm)
    torch.cuda.synchronize()
    reps = P.read_report(o["rep"])
    for k in range(len(lens)):
        a, b = off[k], off[k + 1]
        one = P.pact_reduce(hid[a:b], pre[a:b], ks[a:b], qs[k:k + 1] if mean else qs[a:b], 1, d_h, n_q, prm[k])
        torch.cuda.synchronize()
        rep = P.read_report(one["rep"])
        assert all(reps[k][f] == rep[f] for f in ("n_kept", "n_centers", "n_reincorporated", "zero_norm_seen", "nonfinite_seen", "score_near_ties")), k
        for name, m in (("scores", b - a), ("cluster_id", b - a), ("center_idx", rep["n_centers"]), ("merged", rep["n_centers"]), ("cluster_counts", rep["n_centers"])):
            assert torch.equal(o[name][a:a + m], one[name][:m]), (k, name)


# single samples of more than 90 MB, part of whose norms are in the first launch: hidden states of one and of two launches' rows, rows of a part's end
@pytest.mark.parametrize("n,h,dtype", [(4101, 5600, "f32"), (6403, 3584, "f32"), (11009, 4100, "f32"), (12001, 4096, "bf16")])
def test_norms_in_both_launches(n, h, dtype):
    g = torch.Generator("cuda").manual_seed(n)
    hid = torch.randn(n, h, device="cuda", generator=g).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    ks, qs = (torch.randn(n, 64, device="cuda", generator=g).bfloat16() for _ in range(2))
    assert n * (hid.element_size() * h + 256) > 90e6
    want = hid.double().norm(dim=1) * torch.softmax(ks.double() @ qs.double().mean(0), dim=0)
    for o in (P.pact_score(hid, ks, qs, 1, 64, 1), P.pact_reduce(hid, ks, ks, qs, 1, 64, 1, P.PactParams(0.5, 0.02, 2.0, 1.5))["scores"]):
        torch.cuda.synchronize()
        np.testing.assert_allclose(o[:n].cpu().numpy(), want.cpu().numpy(), rtol=2e-7)
