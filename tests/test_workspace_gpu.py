"""Workspaces smaller than spec_workspace_size() asks for: a launch plan that
takes more than the plain one is dropped where the workspace does not hold it,
so that a workspace of the plain plan's size is enough for every call."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_00722_amd as spec
from tests.gpu_helpers import (SCORE_ABS, SCORE_REL, TOL_ATTN, announce, f64, need_gpu,
                               plain_attn_bytes)
from workloads import generate, generate_mla, small_workload

pytestmark = pytest.mark.gpu

GUARD = 4096


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


def _guarded(nbytes, dev):
    """A workspace of nbytes and the bytes behind it, which must stay as they are."""
    buf = torch.full((nbytes + GUARD,), 0x5A, dtype=torch.uint8, device=dev)
    return buf[:nbytes], buf[nbytes:]


# (n_layers, B, L_cap, H_q, H_kv, counts, k_max): shared units in 32 and 16 parts
# (16 and 8 of the plain plan), and in one (4); launches without partial results
# in either plan, one wavefront per unit (1024 groups) and shared units (400)
ATTN_CASES = [
    (1, 1, 5000, 64, 8, [4096], 4096),
    (1, 2, 2100, 32, 8, [2048, 700], 2048),
    (1, 9, 400, 8, 2, [0, 1, 31, 32, 33, 127, 128, 129, 200], 200),
    (4, 32, 160, 16, 8, [(37 * b) % 129 for b in range(32)], 128),
    (2, 50, 300, 8, 4, [(37 * b) % 201 for b in range(50)], 200),
]


@pytest.mark.parametrize("case", ATTN_CASES, ids=[str(c[:5]) for c in ATTN_CASES])
def test_attention_in_the_plain_workspace(dev, case):
    n_layers, B, L_cap, H_q, H_kv, counts, k_max = case
    announce(f"attn plain workspace {case[:5]}")
    g = torch.Generator(device=dev).manual_seed(3 + sum(case[:5]))
    q, K, V = (torch.randn(s, generator=g, device=dev).to(torch.bfloat16)
               for s in ((n_layers, B, H_q, 128),) + ((n_layers, B, L_cap, H_kv, 128),) * 2)
    rng = np.random.default_rng(5)
    idx = np.full((B, k_max), -1, dtype=np.int32)
    for b in range(B):
        idx[b, :counts[b]] = np.sort(rng.choice(L_cap, counts[b], replace=False))
    ix = torch.as_tensor(idx, device=dev)
    cnt = torch.tensor(counts, dtype=torch.int32, device=dev)
    out = torch.empty((n_layers, B, H_q, 128), device=dev)
    lse = torch.empty((n_layers, B, H_q), device=dev)
    need = plain_attn_bytes(n_layers, B, H_q, H_kv, k_max)
    ws, behind = _guarded(need, dev)
    for o, l in ((out, lse), (None, None)):   # native and ctypes marshalling
        got, gl = spec.sparse_decode_attn(q, K, V, cnt, idx=ix, out=o, lse=l, ws=ws)
        assert bool((behind == 0x5A).all())
        for layer in range(n_layers):
            for b in range(B):
                want, wl = oracle.sparse_gqa_attention(f64(q)[layer, b], f64(K[layer, b]),
                                                       f64(V[layer, b]), idx[b, :counts[b]])
                assert np.abs(got[layer, b].cpu().numpy() - want).max() <= TOL_ATTN, (layer, b)
                if counts[b]:
                    assert np.abs(gl[layer, b].cpu().numpy() - wl).max() <= TOL_ATTN, (layer, b)
    if need:
        with pytest.raises(ValueError):
            spec.sparse_decode_attn(q, K, V, cnt, idx=ix, ws=ws[:need - 16])


# Lengths that leave the logits rows of the plain layout unaligned; one row kernel
# per score row (short rows) and the tiled selection; blocks of 64, 128 and 256
# tokens where the other plan takes fewer or more
STEP_CASES = [
    (dict(B=2, L=1003, H_r=8, d_r=64, n_layers=1, H_q=32, H_kv=8, k=500, ragged_min=3), False),
    (dict(B=1, L=3, H_r=3, d_r=64, n_layers=1, H_q=4, H_kv=1, k=2), False),
    (dict(B=3, L=20001, H_r=16, d_r=64, n_layers=1, H_q=16, H_kv=8, k=600, ragged_min=9000), True),
    (dict(B=150, L=334, H_r=8, d_r=128, n_layers=1, H_q=8, H_kv=2, k=40, ragged_min=1), False),
    (dict(B=40, L=9001, H_r=16, d_r=64, n_layers=1, H_q=4, H_kv=2, k=300, ragged_min=5000), False),
]


@pytest.mark.parametrize("kw,heads", STEP_CASES, ids=[f"B{k['B']}L{k['L']}" for k, _ in STEP_CASES])
def test_step_in_the_plain_workspace(dev, kw, heads):
    announce(f"step plain workspace {kw} heads={heads}")
    w = small_workload(**kw)
    x = generate(w, seed=kw["B"] + kw["L"], device=dev)
    n_sets = w.H_kv if heads else 1
    need = spec.workspace_size(spec.Dims.make(
        B=w.B, L_cap=w.L_cap, L_max=w.L_cap, k_max=w.k, H_r=w.H_r, d_r=w.d_r, n_layers=w.n_layers,
        H_q=w.H_q, H_kv=w.H_kv, d=w.d, n_sets=n_sets), spec.OP_STEP_NOALLOC)
    ws, behind = _guarded(need, dev)
    args = (x["q_r"], x["K_r"], x["seq_lens"], x["ks"], x["q"], x["K"], x["V"], w.k)
    r = spec.step(*args, with_scores=True, with_lse=True, head_level=heads, ws=ws)
    assert bool((behind == 0x5A).all())
    idx, cnt = r["idx"].cpu().numpy(), r["counts"].cpu().numpy()
    sc = r["scores"].cpu().numpy().astype(np.float64)
    q, K, V = (f64(x[n]) for n in ("q", "K", "V"))
    for b in {0, w.B // 2, w.B - 1}:
        L = int(x["seq_lens"][b])
        kb = min(int(x["ks"][b]), L)
        assert cnt[b] == kb
        qr, kr = f64(x["q_r"][b]), f64(x["K_r"][b])
        want = (oracle.head_level_scores(qr, kr, L, n_sets) if heads
                else oracle.retrieval_scores(qr, kr, L)[None])
        got = sc[b] if heads else sc[b][None]
        sets = idx[b] if heads else idx[b][None]
        assert np.all(np.abs(got[:, :L] - want) <= SCORE_ABS + SCORE_REL * want), b
        assert np.all(np.isneginf(got[:, L:])), b
        for g in range(n_sets):
            assert sets[g, :kb].tolist() == oracle.topk_indices(got[g, :L], kb).tolist(), (b, g)
        if heads:
            o, l = oracle.sparse_gqa_attention_sets(q[0, b], K[0, b], V[0, b],
                                                    [s[:kb] for s in sets])
        else:
            o, l = oracle.sparse_gqa_attention(q[0, b], K[0, b], V[0, b], sets[0, :kb])
        assert np.abs(r["out"][0, b].cpu().numpy() - o).max() <= TOL_ATTN, b
        if kb:
            assert np.abs(r["lse"][0, b].cpu().numpy() - l).max() <= TOL_ATTN, b
    with pytest.raises(ValueError):
        spec.step(*args, head_level=heads, ws=ws[:need - 16])


def plain_mla_bytes(n_layers, B, H, k_max):
    """The least MLA workspace: absorbed queries and the partial results of
    splits of 256 to 2048 tokens, at most 16 a sequence, that make 256 units."""
    ceil = lambda a, b: -(-a // b)
    al = lambda n: ceil(n, 256) * 256
    split = ceil(ceil(k_max, min(16, ceil(256, n_layers * B * (H // 64)))), 32) * 32
    units = n_layers * B * ceil(k_max, min(max(split, 256), 2048))
    return al(2 * n_layers * B * H * (2 * 512 + 64)) + al(4 * units * H * 512) + al(8 * units * H)


# Launches cut into more splits than the plain plan's, and into fewer
@pytest.mark.parametrize("case", [(1, 1, 700, 128), (1, 4, 1000, 64), (8, 9, 300, 128)],
                         ids=["l1_B1", "l1_B4", "l8_B9"])
def test_mla_in_the_plain_workspace(dev, case):
    n_layers, B, k, H = case
    announce(f"mla plain workspace {case}")
    w = small_workload(B=B, L=k + 50, k=k, n_layers=n_layers, H_q=H, H_kv=1, mla=True)
    x = generate_mla(w, seed=29, device=dev)
    counts = [k - 30 * b for b in range(B)]
    rng = np.random.default_rng(31)
    idx = np.full((B, k), -1, dtype=np.int32)
    for b in range(B):
        idx[b, :counts[b]] = np.sort(rng.choice(k + 50, counts[b], replace=False))
    args = (x["q_mla"], x["ckv"], x["w_uk"], x["w_uv"], torch.as_tensor(idx, device=dev),
            torch.tensor(counts, dtype=torch.int32, device=dev))
    need = plain_mla_bytes(n_layers, B, H, k)
    ws, behind = _guarded(need, dev)
    out = torch.empty((n_layers, B, H, 128), device=dev)
    for o in (out, None):   # native and ctypes marshalling
        got, _ = spec.mla_sparse_decode_attn(*args, out=o, with_lse=False, ws=ws)
        assert bool((behind == 0x5A).all())
        for b in {0, B - 1}:
            heads = [0, 17, H - 1]
            q, c = f64(x["q_mla"][-1, b])[heads], f64(x["ckv"][-1, b])
            want, _ = oracle.mla_sparse_attention(
                q[:, :128], q[:, 128:], c[:, :512], c[:, 512:], f64(x["w_uk"][-1])[heads],
                f64(x["w_uv"][-1])[heads], idx[b, :counts[b]])
            assert np.abs(got[-1, b].cpu().numpy()[heads] - want).max() <= TOL_ATTN, b
    with pytest.raises(ValueError):
        spec.mla_sparse_decode_attn(*args, ws=ws[:need - 16])
