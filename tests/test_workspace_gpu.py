"""Workspaces smaller than spec_workspace_size() asks for: a launch plan that
takes more than the plain one is dropped where the workspace does not hold it,
so that a workspace of the plain plan's size is enough for every call."""
import numpy as np
import pytest
import torch

import oracle
import paper_2512_00722_amd as spec
from tests.gpu_helpers import TOL_ATTN, announce, f64, need_gpu, plain_attn_bytes

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
