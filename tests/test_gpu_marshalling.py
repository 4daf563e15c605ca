"""The two ways into the C entry points -- the C++ marshalling and the ctypes path it leaves irregular arguments to -- launch the
same work, and refuse the same calls."""
import pytest
import torch

import paper_2412_05496_amd as fa
from paper_2412_05496_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


class Params(fa.ModParams):      # a subclass goes the ctypes way
    pass


def outputs(params_type):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    r = lambda *s: torch.randn(*s, generator=gen, dtype=torch.bfloat16, device=DEV)
    out = []
    docs = (torch.arange(320, device=DEV, dtype=torch.int32) // 70).repeat(2, 1)
    p = params_type(window=50, prefix_len=7, softcap=20, doc_ids=docs, alibi_bias=-torch.rand(4, generator=gen, device=DEV),
                    rel_bias=torch.randn(4, 33, generator=gen, device=DEV))
    Q, dO = (r(2, 320, 4, 64).transpose(1, 2) for _ in range(2))           # [B, S, H, D] in memory
    K, V = r(2, 2, 320, 64), r(2, 2, 320, 64)
    for mask, score, Bm in ((fa.MASK_DOCUMENT_CAUSAL, fa.SCORE_REL_BIAS | fa.SCORE_SOFTCAP, 2), (fa.MASK_SWA_CAUSAL_OR_PREFIX, fa.SCORE_REL_BIAS, 1),
                            (fa.MASK_CAUSAL, fa.SCORE_ALIBI, 1)):
        bm = fa.alloc_blockmask(Bm, 1, 320, 320, 128, 64, device=DEV)
        fa.flexattn_blockmask_build(mask, p, bm)
        O, L = torch.empty_like(Q), torch.empty(2, 4, 320, device=DEV)
        fa.flexattn_forward(Q, K, V, score, mask, p, bm, 0.125, O, L)
        g = [torch.empty_like(t) for t in (Q, K, V)] + [torch.empty_like(t) for t in (Q, K, V)]
        fa.flexattn_backward(Q, K, V, O, dO, L, score, mask, p, bm, 0.125, *g[:3])
        fa.flexattn_backward_stored(Q, K, V, O, dO, L, score, mask, p, bm, 0.125, *g[3:], int(bm.stats[:2].sum()))
        out += [O, L, *g, bm.kv_indices, bm.full_kv_indices, bm.q_order, bm.stats]
    pool_k, pool_v = r(9, 2, 64, 64), r(9, 2, 64, 64)
    table = torch.tensor([[3, 1, 7, 0], [2, 8, 4, 5]], dtype=torch.int32, device=DEV)
    ctx = torch.tensor([200, 131], dtype=torch.int32, device=DEV)
    q1 = r(2, 4, 1, 64)
    ws = torch.empty(max(16, fa.flexattn_paged_decode_workspace_bytes(q1, pool_k, table)), dtype=torch.uint8, device=DEV)
    o1, l1 = torch.empty(2, 4, 64, dtype=torch.bfloat16, device=DEV), torch.empty(2, 4, device=DEV)
    for mask in (fa.MASK_CTX_LEN, fa.MASK_CTX_LEN_WINDOW):
        for lse in (l1, None):
            fa.flexattn_paged_decode(q1, pool_k, pool_v, table, ctx, fa.SCORE_ALIBI, mask, p, 0.125, o1, lse, ws)
            out += [o1.clone(), l1.clone()]
    chunk = params_type(q_offsets=torch.tensor([100, 31], dtype=torch.int32, device=DEV))
    Qc = r(2, 4, 100, 64)
    bm = fa.alloc_blockmask(2, 1, 100, 256, 128, 64, device=DEV)
    fa.flexattn_blockmask_build(fa.MASK_CAUSAL, chunk, bm)
    phys, full = torch.zeros_like(bm.kv_indices), torch.zeros_like(bm.full_kv_indices)
    back = torch.full((9,), -1, dtype=torch.int32, device=DEV)
    fa.flexattn_paged_convert_blockmask(bm.kv_num_blocks, bm.kv_indices, table, phys, back)
    fa.flexattn_paged_convert_blockmask(bm.full_kv_num_blocks, bm.full_kv_indices, table, full)
    Oc, Lc = torch.empty_like(Qc), torch.empty(2, 4, 100, device=DEV)
    fa.flexattn_paged_forward(Qc, pool_k, pool_v, fa.SCORE_IDENTITY, fa.MASK_CAUSAL, chunk, bm, phys, full, 0.125, Oc, Lc)
    return out + [phys, full, back, Oc, Lc]


def test_both_paths_do_the_same():
    assert hasattr(binding._fast(), "setup"), "csrc/marshal.cpp has not been built"
    for i, (a, b) in enumerate(zip(outputs(fa.ModParams), outputs(Params))):
        assert torch.equal(a, b), i
    torch.cuda.synchronize()


@pytest.mark.parametrize("params_type", [fa.ModParams, Params])
def test_both_paths_refuse_the_same(params_type):
    z = lambda *s, dtype=torch.bfloat16: torch.zeros(*s, dtype=dtype, device=DEV)
    Q, L, p = z(1, 2, 128, 64), z(1, 2, 128, dtype=torch.float32), params_type()
    bm = fa.alloc_blockmask(1, 1, 128, 128, 128, 64, device=DEV)
    fa.flexattn_blockmask_build(fa.MASK_CAUSAL, p, bm)
    fwd = lambda **k: fa.flexattn_forward(*[{**dict(Q=Q, K=Q, V=Q, score_id=0, mask_id=fa.MASK_CAUSAL, params=p, bm=bm, scale=0.1, O=Q.clone(), LSE=L),
                                             **k}[n] for n in ("Q", "K", "V", "score_id", "mask_id", "params", "bm", "scale", "O", "LSE")])
    fwd()
    for bad in (dict(Q=z(1, 2, 128, 64, dtype=torch.float16)), dict(K=Q.cpu()), dict(O=Q.transpose(2, 3)), dict(LSE=L.double()), dict(LSE=L[:, :1]),
                dict(params=params_type(alibi_bias=z(2)))):
        with pytest.raises(AssertionError):
            fwd(**bad)
    for bad in (dict(scale=-1.0), dict(score_id=fa.SCORE_ALIBI), dict(mask_id=77), dict(Q=Q[..., :32], K=Q[..., :32], V=Q[..., :32])):
        with pytest.raises(fa.FlexAttnError):
            fwd(**bad)
    with pytest.raises(Exception):
        fwd(scale="0.1")
    with pytest.raises(fa.FlexAttnError):
        fa.flexattn_blockmask_build(fa.MASK_DOCUMENT, p, bm)
    torch.cuda.synchronize()
