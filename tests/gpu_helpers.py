"""Shared glue for the GPU parity tests (no method arithmetic here)."""
import os
import sys

import numpy as np
import pytest
import torch

TOL_ATTN = 2e-3          # max-abs on attention outputs (bf16 in, fp32 accumulate)
SCORE_ABS, SCORE_REL = 1e-7, 1e-5   # internal gate on retrieval scores


def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU on this host")
    import paper_2512_00722_amd as spec
    spec.load_library()   # raises if the HIP library is missing: no fallback exists
    return torch.device("cuda:0")


def f64(t: torch.Tensor) -> np.ndarray:
    """Exact float64 copy of a (bf16 / fp32) tensor."""
    return t.detach().float().cpu().numpy().astype(np.float64)


def announce(msg: str):
    print(f"[case] {msg}", flush=True)
    sys.stdout.flush()


def plain_attn_bytes(n_layers, B, H_q, H_kv, k_max) -> int:
    """The least attention workspace: partial results with one wavefront per
    unit (at most 1024 units of 256 to 2048 tokens, 64 where units of 256 would
    be fewer than 64), in two regions of whole 256 bytes."""
    ceil = lambda a, b: -(-a // b)
    groups = n_layers * B * H_kv * max(1, H_q // H_kv // 16)
    least = 64 if groups * ceil(k_max, 256) < 64 else 256
    split = min(max(ceil(ceil(k_max, ceil(1024, groups)), 32) * 32, least), 2048)
    n = ceil(k_max, split)
    rows = n_layers * B * n * H_q
    return 0 if n == 1 else ceil(rows * 512, 256) * 256 + ceil(rows * 8, 256) * 256
