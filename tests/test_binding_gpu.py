"""The binding's native marshalling (calls that hand over every buffer)
against its ctypes path: the same bits, the same errors, and what the ctypes
path accepts or refuses beyond it stays accepted or refused."""
import pytest
import torch

import paper_2512_00722_amd as spec
from tests.gpu_helpers import announce, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return need_gpu()


class Sub(torch.Tensor):
    """A tensor subclass: never plain."""


def _case(dev, heads=False, layers=2):
    g = torch.Generator(device=dev).manual_seed(5)
    B, L, k, H_r, H_q, H_kv = 3, 700, 150, 8, 16, 4

    def rn(*shape):
        return torch.randn(shape, generator=g, device=dev).to(torch.bfloat16)

    def i32(*v):
        return torch.tensor(v, dtype=torch.int32, device=dev)

    return dict(q_r=rn(B, H_r, 64), K_r=rn(B, L, H_r, 64), lens=i32(700, 0, 333),
                ks=i32(150, 10, 83), q=rn(layers, B, H_q, 128), K=rn(layers, B, L, H_kv, 128),
                V=rn(layers, B, L, H_kv, 128), k=k, B=B, L=L, H_q=H_q, H_kv=H_kv, layers=layers)


def _ws(dev, n=1 << 25):
    return torch.empty(n, dtype=torch.uint8, device=dev)


def _step_outputs(c, dev, heads, scores=True):
    sets = (c["H_kv"],) if heads else ()
    n, B = c["layers"], c["B"]
    return dict(idx=torch.empty((B,) + sets + (c["k"],), dtype=torch.int32, device=dev),
                counts=torch.empty((B,), dtype=torch.int32, device=dev),
                out=torch.empty((n, B, c["H_q"], 128), device=dev),
                lse=torch.empty((n, B, c["H_q"]), device=dev),
                scores=torch.empty((B,) + sets + (c["L"],), device=dev) if scores else None)


@pytest.mark.parametrize("heads", [False, True], ids=["one_set", "head_sets"])
def test_step_native_equals_ctypes(dev, heads):
    announce(f"binding step heads={heads}")
    c = _case(dev)
    a = [c[n] for n in ("q_r", "K_r", "lens", "ks", "q", "K", "V", "k")]
    want = spec.step(*a, with_scores=True, with_lse=True, head_level=heads)
    got = _step_outputs(c, dev, heads)
    assert spec.step(*a, outputs=got, ws=_ws(dev), head_level=heads) is got
    assert spec._fast.step(*a, None, 0.0, 0.0, None, got, heads, _ws(dev),
                           spec._raw_stream(c["q"])) == 0   # the native path takes it
    for n in ("idx", "counts", "out", "lse", "scores"):
        assert torch.equal(want[n], got[n]), n
    if not heads:   # elastic, with a clamped row limit
        s1, s2 = (spec.ElasticState(c["layers"], c["B"], c["k"], c["H_kv"], 128, dev)
                  for _ in range(2))
        w = spec.step(*a, L_max=650, elastic=s1, with_lse=True)
        o = _step_outputs(c, dev, False, scores=False)
        spec.step(*a, L_max=650, elastic=s2, outputs=o, ws=_ws(dev))
        for n in ("idx", "counts", "out", "lse"):
            assert torch.equal(w[n], o[n]), n
        for n in ("slot_tok", "slot_src", "n_changed", "kbuf", "vbuf"):
            assert torch.equal(getattr(s1, n), getattr(s2, n)), n


def test_ops_native_equal_ctypes(dev):
    announce("binding ops")
    c = _case(dev)
    ws = _ws(dev)
    sc = spec.score(c["q_r"], c["K_r"], c["lens"], n_sets=4)
    assert torch.equal(sc, spec.score(c["q_r"], c["K_r"], c["lens"], out=torch.empty_like(sc),
                                      ws=ws, n_sets=4))
    idx, counts = spec.topk(sc, c["lens"], c["ks"], c["k"])
    i2, c2 = spec.topk(sc, c["lens"], c["ks"], c["k"], idx=torch.empty_like(idx),
                       counts=torch.empty_like(counts), ws=ws)
    assert torch.equal(idx, i2) and torch.equal(counts, c2)
    # strided caches: every other layer of a longer cache
    K = c["K"].repeat(2, 1, 1, 1, 1)[::2]
    V = c["V"].repeat(2, 1, 1, 1, 1)[::2]
    for ix in (idx, None):
        kk, vv = (K, V) if ix is not None else (c["K"], c["V"])
        out, lse = spec.sparse_decode_attn(c["q"], kk, vv, counts, idx=ix, scale=0.07)
        o2, l2 = spec.sparse_decode_attn(c["q"], kk, vv, counts, idx=ix, scale=0.07,
                                         out=torch.empty_like(out), lse=torch.empty_like(lse),
                                         ws=ws)
        assert torch.equal(out, o2) and torch.equal(lse, l2)
    g = torch.Generator(device=dev).manual_seed(6)

    def rn(*shape):
        return torch.randn(shape, generator=g, device=dev).to(torch.bfloat16)

    m = (rn(1, 3, 64, 192), rn(1, 3, 400, 576), rn(1, 64, 128, 512), rn(1, 64, 128, 512),
         idx[:, 0].contiguous().clamp(max=399), counts)
    out, lse = spec.mla_sparse_decode_attn(*m)
    o2, none = spec.mla_sparse_decode_attn(*m, out=torch.empty_like(out), with_lse=False, ws=ws)
    assert torch.equal(out, o2) and none is None
    f = (torch.tensor([5, 99, 2], dtype=torch.int32, device=dev),
         torch.tensor([0, 699, 700], dtype=torch.int32, device=dev), rn(100, 256),
         rn(512, 256), rn(512, 256))
    k1, k2 = c["K_r"].clone(), c["K_r"].clone()
    q1 = spec.retrieval_qk(*f, k1, yarn_scale=4.0)
    q2 = spec.retrieval_qk(*f, k2, yarn_scale=4.0, q_r=torch.empty_like(q1), ws=ws)
    assert torch.equal(q1, q2) and torch.equal(k1, k2)


def test_refused_and_accepted(dev):
    announce("binding errors")
    c = _case(dev)
    ws, idx = _ws(dev), torch.zeros((3, 150), dtype=torch.int32, device=dev)
    counts = torch.tensor([150, 0, 9], dtype=torch.int32, device=dev)
    out = torch.empty((2, 3, 16, 128), device=dev)
    lse = torch.empty((2, 3, 16), device=dev)

    def attn(q=c["q"], K=c["K"], V=c["V"], counts=counts, out=out, lse=lse, ws=ws, **kw):
        return spec.sparse_decode_attn(q, K, V, counts, idx=idx, out=out, lse=lse, ws=ws, **kw)

    attn()
    want = out.clone()
    for kw, err in ((dict(q=c["q"].float()), TypeError), (dict(counts=counts.long()), TypeError),
                    (dict(q=c["q"][0]), ValueError), (dict(q=c["q"].cpu()), ValueError),
                    (dict(V=c["V"][:, :, :-1]), ValueError), (dict(K=1), TypeError),
                    (dict(counts=counts[:2]), ValueError), (dict(ws=ws[:16]), None),
                    (dict(scale=-1.0), spec.SpecError),
                    (dict(scale=float("nan")), spec.SpecError)):
        if err is None:   # no workspace is needed: a small one is enough
            need = spec.workspace_size(spec.Dims.make(3, 700, 700, 150, n_layers=2, H_q=16,
                                                      H_kv=4), spec.OP_ATTN)
            if need <= 16:
                attn(**kw)
                continue
            err = ValueError
        with pytest.raises(err):
            attn(**kw)
    with pytest.raises(ValueError):   # the step's workspace
        o = _step_outputs(c, dev, False)
        spec.step(*[c[n] for n in ("q_r", "K_r", "lens", "ks", "q", "K", "V", "k")], outputs=o,
                  ws=ws[:64])
    # unusual but accepted: a flat output, a subclass, an integer scale
    flat = torch.empty(out.numel(), device=dev)
    attn(out=flat)
    assert torch.equal(flat.view(out.shape), want)
    out.zero_()
    attn(q=c["q"].as_subclass(Sub), scale=0)
    assert torch.equal(out, want)
    # batched tensors have no memory of their own: refused as before
    with pytest.raises(RuntimeError):
        torch.vmap(lambda q: attn(q=q)[0])(c["q"][None])


def test_current_stream(dev):
    """The call goes to the current stream, also with native marshalling."""
    announce("binding stream")
    c = _case(dev)
    s = torch.cuda.Stream()
    o = _step_outputs(c, dev, False)
    a = [c[n] for n in ("q_r", "K_r", "lens", "ks", "q", "K", "V", "k")]
    ws = _ws(dev)
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        assert spec._raw_stream(c["q"]) == s.cuda_stream
        spec.step(*a, outputs=o, ws=ws)
    s.synchronize()
    want = spec.step(*a, with_lse=True)
    assert torch.equal(want["out"], o["out"])
