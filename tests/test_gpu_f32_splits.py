"""GPU parity of the float32 path where its split sums have edges: the dH vocabulary split (one
workgroup tile and many, a vocabulary of one, of one split step more or less, ragged last split) and
the float32 LoRA passes (row and column remainders of their 16-wide chunks, several rank tiles)
against the float64 oracle. Bound 1e-5 normwise, the float32 bar of the other parity tests: sums of at
most 5000 float32 products in blocks of at least four partial sums."""
import numpy as np
import pytest

from gpu_util import dev_dense, dev_f32, dev_i32, host, note, rel_norm
from oracle import ce as oce
from oracle import lora as olora
from workloads.gen import random_dense

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.mark.parametrize("N,d,V", [(1, 8, 1), (3, 8, 127), (64, 64, 128), (65, 72, 129), (63, 136, 2049),
                                   (200, 256, 4097), (513, 1024, 700), (2048, 1032, 300)])
def test_ce_f32_splits(attt, N, d, V):
    note(f"ce f32 N={N} d={d} V={V}")
    rng = np.random.default_rng(N + d + V)
    h, W = random_dense((N, d), 1.0, False, 5), random_dense((V, d), 0.05, False, 6)
    labels, w = rng.integers(0, V, N), rng.uniform(0.05, 1, N).astype(np.float32)
    off = np.array([0, N // 3, N], np.int64)
    loss, lse, dH = (host(t) for t in attt.weighted_ce_fwd_bwd(dev_dense(h), dev_dense(W), dev_i32(labels), dev_f32(w),
                                                               row_offsets=off))
    lo, lseo, dHo = oce.weighted_ce(h.f32, W.f32, labels, w, off)
    if V > 1:  # one class: loss and gradient are 0 up to rounding
        assert np.all(np.abs(loss - lo) <= TOL * (np.abs(lo) + 1e-3))
        assert rel_norm(dH, dHo) <= TOL
    else:
        assert np.max(np.abs(dH)) <= 1e-6 and np.max(np.abs(loss)) <= 1e-6
    assert np.max(np.abs(lse - lseo) / (1e-2 + np.abs(lseo))) <= TOL


@pytest.mark.parametrize("rows,d_in,d_out,ranks", [(1, 8, 8, (1,)), (15, 24, 72, (16,)), (129, 64, 136, (17, 8)),
                                                   (512, 264, 256, (8, 33)), (2100, 256, 512, (64,))])
def test_lora_f32_remainders(attt, rows, d_in, d_out, ranks):
    import torch
    note(f"lora f32 rows={rows} {d_in}->{d_out} ranks {ranks}")
    x = random_dense((rows, d_in), 1.0, False, 7)
    tx, probs, refs = dev_dense(x), [], []
    for i, r in enumerate(ranks):  # one x: the problems share a job
        dy, A, B = (random_dense(s, 0.1, False, 11 * i + k) for k, s in enumerate([(rows, d_out), (r, d_in), (d_out, r)]))
        probs.append(dict(x=tx, dy=dev_dense(dy), A=dev_dense(A), B=dev_dense(B), scale=2.0,
                          dA=torch.zeros(r, d_in, device="cuda"), dB=torch.zeros(d_out, r, device="cuda")))
        refs.append(olora.lora_grad(x.f32, dy.f32, A.f32, B.f32, 2.0))
    attt.lora_grad(probs)
    for p, (dA, dB) in zip(probs, refs):
        assert rel_norm(host(p["dA"]), dA) <= TOL and rel_norm(host(p["dB"]), dB) <= TOL


@pytest.mark.parametrize("V", [1, 33, 64, 65, 97, 128, 161])
@pytest.mark.parametrize("bad", ["nan", "-inf", "mixed", "inf"])
def test_ce_f32_head_rows_not_finite(attt, V, bad):
    """Non-finite logits in the last head row, in its whole block of 32 and in all of them: a NaN or +inf
    logit makes the loss, lse and dH of every token NaN; -inf logits have probability 0. (lse within the
    float32 bar of this file.)"""
    import torch
    note(f"ce f32 V={V} {bad}")
    N, d = 5, 8
    g = torch.Generator()
    g.manual_seed(V)
    # positive hidden states and one head entry of 1 in the rows' column 0: the logit is h_0 times that entry
    h = torch.rand(N, d, generator=g) + 0.5
    labels, w = torch.zeros(N, dtype=torch.int32), torch.ones(N)
    for first in sorted({V - 1, (V - 1) // 32 * 32, 0}):
        W = torch.randn(V, d, generator=g) * 0.1
        W[first:] = 0.0
        W[first:, 0] = float(bad) if bad != "mixed" else float("-inf")
        if bad == "mixed":
            W[V - 1, 0] = float("nan")
        for grad in (False, True):
            loss, lse, dH = attt.weighted_ce_fwd_bwd(h.cuda(), W.cuda(), labels.cuda(), w.cuda(), want_grad=grad)
            if bad == "-inf":
                z = h.double() @ torch.where(torch.isinf(W), 0.0, W).double().t()
                z[:, first:] = float("-inf")
                assert torch.allclose(lse.cpu().double(), torch.logsumexp(z, 1), rtol=TOL, atol=TOL)
                assert torch.isnan(loss).all() == (first == 0)  # the label's logit is -inf too
            else:
                assert torch.isnan(loss).all() and torch.isnan(lse).all(), (first, loss, lse)
                assert dH is None or torch.isnan(dH).any(1).all()
