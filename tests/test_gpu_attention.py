"""GPU parity of the adapted attention block's backward (dY_q = dQ, dY_k = dK, dY_v = dV; the
upstream gradients of the q/k/v LoRA gradient) against the float64 oracle, on the same bf16
inputs: every row's cosine >= 0.999 and every element within 2^-7 (|ref| + rms of its row),
lse and D (the forward statistics the kernels also return) to float32 accuracy.

Shapes: small ragged episodes (one-row episode, exact and partial 64-row blocks), grouped-head
ratios 1, 2, 4 and 8, the small workload's shape (2048 rows, 16 heads over 4 key/value heads)
in full, the Llama-8B shape (8192 rows, 32 heads over 8) with the oracle on one key/value
group, and 16 episodes of 4096 rows with the oracle on two episodes."""
import numpy as np
import pytest

from gpu_util import check_rows, cosine, dev_dense, host, note
from oracle import attention as oat
from workloads.gen import random_dense

pytestmark = pytest.mark.gpu
DH = 128
BF16_COS = 0.999
BF16_ELEM = 2.0 ** -7


def _inputs(N, H, Hkv, seed):
    q = random_dense((N, H, DH), 1.0, True, seed)
    k = random_dense((N, Hkv, DH), 1.0, True, seed + 1)
    v = random_dense((N, Hkv, DH), 1.0, True, seed + 2)
    do = random_dense((N, H, DH), 0.05, True, seed + 3)
    return q, k, v, do


def _gpu(attt, q, k, v, do, off):
    dq, dk, dv, lse, dsum = attt.attention_bwd(dev_dense(q), dev_dense(k), dev_dense(v), dev_dense(do), row_offsets=off)
    return host(dq), host(dk), host(dv), lse.cpu().numpy(), dsum.cpu().numpy()


def _cmp(name, got, want):
    g2, w2 = got.reshape(got.shape[0], -1), want.reshape(want.shape[0], -1)
    live = np.linalg.norm(w2, axis=1) > 0
    assert cosine(g2, w2) >= BF16_COS, name
    check_rows(g2[live], w2[live], BF16_COS, BF16_ELEM, name)
    # rows whose exact gradient is 0 (an episode's first query: one key, so dS = 0; a key no later
    # query of its episode sees) are negligible against the tensor's scale: dP and D round in
    # different orders, so dP - D is tiny but not always exactly 0
    if np.any(~live):
        assert np.max(np.abs(g2[~live])) <= BF16_ELEM * np.sqrt(np.mean(w2 ** 2)), name


def _check_full(attt, N, H, Hkv, off, seed):
    q, k, v, do = _inputs(N, H, Hkv, seed)
    dq, dk, dv, lse, dsum = _gpu(attt, q, k, v, do, off)
    r = oat.attention_fwd_bwd(q.f32, k.f32, v.f32, do.f32, off)
    _cmp("dQ", dq, r["dQ"])
    _cmp("dK", dk, r["dK"])
    _cmp("dV", dv, r["dV"])
    assert np.max(np.abs(lse - r["lse"])) <= 1e-4 * (1 + np.max(np.abs(r["lse"])))
    assert np.max(np.abs(dsum - r["D"])) <= 1e-3 * (1e-6 + np.sqrt(np.mean(r["D"] ** 2)))


@pytest.mark.parametrize("H,Hkv", [(4, 4), (4, 2), (8, 2), (8, 1)])
def test_small_ragged(attt, H, Hkv):
    off = np.array([0, 1, 65, 129, 200, 264, 300], np.int64)
    note(f"attention small ragged: heads {H}/{Hkv}, episodes {np.diff(off).tolist()}")
    _check_full(attt, int(off[-1]), H, Hkv, off, 11 + H + Hkv)


def test_single_episode_no_offsets(attt):
    q, k, v, do = _inputs(130, 2, 1, 21)
    dq, dk, dv, lse, dsum = _gpu(attt, q, k, v, do, None)
    r = oat.attention_fwd_bwd(q.f32, k.f32, v.f32, do.f32, None)
    _cmp("dQ", dq, r["dQ"])
    _cmp("dK", dk, r["dK"])
    _cmp("dV", dv, r["dV"])


def test_small_workload_shape(attt):
    note("attention 2048 rows, 16/4 heads")
    _check_full(attt, 2048, 16, 4, np.array([0, 2048], np.int64), 31)


def test_llama8b_shape_one_group(attt):
    N, H, Hkv, g = 8192, 32, 8, 4
    q, k, v, do = _inputs(N, H, Hkv, 41)
    note("attention 8192 rows, 32/8 heads (oracle: key/value head 3 and its 4 query heads)")
    dq, dk, dv, lse, dsum = _gpu(attt, q, k, v, do, None)
    kh = 3
    sl = slice(kh * g, (kh + 1) * g)
    r = oat.attention_fwd_bwd(q.f32[:, sl], k.f32[:, kh:kh + 1], v.f32[:, kh:kh + 1], do.f32[:, sl], None)
    _cmp("dQ", dq[:, sl], r["dQ"])
    _cmp("dK", dk[:, kh:kh + 1], r["dK"])
    _cmp("dV", dv[:, kh:kh + 1], r["dV"])
    assert np.max(np.abs(lse[sl] - r["lse"])) <= 1e-4 * (1 + np.max(np.abs(r["lse"])))


def test_many_episodes_two_checked(attt):
    E, Lr, H, Hkv = 16, 4096, 8, 2
    off = np.arange(E + 1, dtype=np.int64) * Lr
    q, k, v, do = _inputs(E * Lr, H, Hkv, 51)
    note("attention 16 episodes x 4096 rows, 8/2 heads (oracle on episodes 0 and 15)")
    dq, dk, dv, lse, dsum = _gpu(attt, q, k, v, do, off)
    for e in (0, E - 1):
        rs = slice(off[e], off[e + 1])
        r = oat.attention_fwd_bwd(q.f32[rs], k.f32[rs], v.f32[rs], do.f32[rs], None)
        _cmp(f"dQ ep{e}", dq[rs], r["dQ"])
        _cmp(f"dK ep{e}", dk[rs], r["dK"])
        _cmp(f"dV ep{e}", dv[rs], r["dV"])


@pytest.mark.parametrize("H,wide", [(16, False), (32, True)])
def test_one_or_two_query_tiles_per_wave(attt, H, wide):
    """Workgroups of 64 and of 128 queries (more than 768 of the latter): episodes that end inside the
    first and the second half of a 128-query block, on its edges and on those of a wave's 32 queries."""
    lens = [1, 31, 33, 63, 64, 65, 97, 127, 128, 129, 191, 192, 193, 200, 256, 257, 130]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    assert (sum((n + 127) // 128 for n in lens) * H > 768) == wide
    note(f"attention ragged: {H} heads, episodes {lens}")
    _check_full(attt, int(off[-1]), H, 4, off, 71)


def _no_workspace(attt, q, k, v, do, off):
    """The C entry point that takes no workspace: one workgroup per key block."""
    import ctypes

    import torch
    N, H, _ = q.shape
    out = [torch.empty_like(q), torch.empty_like(k), torch.empty_like(v), torch.empty(H, N, device="cuda"),
           torch.empty(H, N, device="cuda")]
    st = attt.load().attt_attention_bwd(*[t.data_ptr() for t in (q, k, v, do)],
                                        off.ctypes.data_as(ctypes.POINTER(ctypes.c_int64)), len(off) - 1, N, H,
                                        k.shape[1], DH, 1.0 / DH ** 0.5, *[t.data_ptr() for t in out],
                                        torch.cuda.current_stream().cuda_stream)
    assert st == attt.OK
    return out


@pytest.mark.parametrize("lens,H,Hkv", [([1, 63, 64, 65, 127, 128, 129, 200] * 9, 8, 8), ([30] * 70, 32, 4),
                                        ([512, 300, 700] * 4, 32, 16)])
def test_many_short_walks(attt, lens, H, Hkv):
    """Batches whose walks are short run in small workgroups, two per CU (the first two choose them, the
    last sits near the line): edges of the 64-row blocks, more episodes than one launch holds."""
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    N = int(off[-1])
    note(f"attention short walks: {len(lens)} episodes, heads {H}/{Hkv}")
    assert attt.attention_workspace_size(N, H, Hkv, off) == 0
    _check_full(attt, N, H, Hkv, off, 91)


def test_no_memory_for_the_workspace(attt):
    """Where the workspace cannot be allocated the block runs unsplit: bitwise attt_attention_bwd's result."""
    import torch
    off = np.array([0, 2048], np.int64)
    q, k, v, do = (dev_dense(t) for t in _inputs(2048, 8, 2, 85))
    assert attt.attention_workspace_size(2048, 8, 2, off) > 20 << 20  # no cached block holds it
    want = _no_workspace(attt, q, k, v, do, off)
    out = tuple(torch.empty_like(t) for t in want)
    torch.cuda.empty_cache()
    torch.cuda.set_per_process_memory_fraction(1e-9)
    try:
        attt.attention_bwd(q, k, v, do, off, out=out)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert all(torch.equal(a, b) for a, b in zip(out, want))


@pytest.mark.parametrize("lens,H,Hkv", [([1, 64, 65, 127, 128, 129], 4, 2), ([700], 8, 1), ([257, 1100, 1, 383], 8, 2),
                                        ([1024], 16, 1), ([33 * 64], 8, 8), ([3000, 64, 2000], 8, 4)])
def test_split_walks(attt, lens, H, Hkv):
    """dK and dV by parts of the queries (whole pieces and rests; a walk of whole pieces alone) and by one
    walk per key block, against the oracle."""
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    N = int(off[-1])
    note(f"attention split: heads {H}/{Hkv}, episodes {lens}, workspace {attt.attention_workspace_size(N, H, Hkv, off)}")
    q, k, v, do = _inputs(N, H, Hkv, 81)
    one = [host(t) for t in _no_workspace(attt, *[dev_dense(t) for t in (q, k, v, do)], off)]
    got = _gpu(attt, q, k, v, do, off)
    r = oat.attention_fwd_bwd(q.f32, k.f32, v.f32, do.f32, off)
    for name, g, o in zip(("dQ", "dK", "dV"), got, one):
        _cmp(name, g, r[name])
        _cmp(name + " (one walk)", o, r[name])
    if sum(lens) > 650:
        assert attt.attention_workspace_size(N, H, Hkv, off) > 0


def test_deterministic(attt):
    q, k, v, do = _inputs(1000, 8, 2, 61)
    off = np.array([0, 300, 1000], np.int64)
    a = _gpu(attt, q, k, v, do, off)
    b = _gpu(attt, q, k, v, do, off)
    for x, y in zip(a, b):
        assert x.tobytes() == y.tobytes()
