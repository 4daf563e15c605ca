"""A launch counts its work items in 32 bits: 2^24 workgroups of 256 are too many, twice as many of 128 are not.  Rows of blocks
of 64 in such numbers (one query each, the same for all, K and V of one head)."""
import pytest
import torch

from oracle import flex_oracle as fo
from tests import helpers as hp

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
HEADS = 2 ** 24 + 24


def problem(D, kv_len, score, seed):
    import paper_2412_05496_amd as fa
    gen = torch.Generator().manual_seed(seed)
    Q, K, V, dO = (torch.randn(1, 1, n, D, generator=gen).to(torch.bfloat16) for n in (1, kv_len, kv_len, 1))
    params = fa.ModParams(q_offsets=torch.tensor([kv_len - 1], dtype=torch.int32, device=DEV))
    if score == "alibi":
        params.alibi_bias = torch.full((HEADS,), -0.01, device=DEV)
    bm = fa.alloc_blockmask(1, 1, 1, kv_len, 64, 64, device=DEV)
    fa.flexattn_blockmask_build(fa.MASK_CAUSAL, params, bm)
    many = [Q.to(DEV).expand(1, HEADS, 1, D), K.to(DEV), V.to(DEV), dO.to(DEV).expand(1, HEADS, 1, D)]
    return (Q, K, V, dO), many, params, bm


def test_forward():
    import paper_2412_05496_amd as fa
    (Q, K, V, _), (q, k, v, _), params, bm = problem(64, 65, "identity", 1)
    print("[case] forward", flush=True)
    O, LSE = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device=DEV), torch.full(q.shape[:3], float("nan"), device=DEV)
    fa.flexattn_forward(q, k, v, fa.SCORE_IDENTITY, fa.MASK_CAUSAL, params, bm, 0.125, O, LSE)
    torch.cuda.synchronize()
    hp.check_output(O[:, :1], LSE[:, :1], *fo.flex_attention(Q, K, V, fo.Identity(), fo.no_mask, 0.125))
    assert torch.equal(O, O[:, :1].expand_as(O)) and torch.equal(LSE, LSE[:, :1].expand_as(LSE))


def test_paged_forward():
    import paper_2412_05496_amd as fa
    (Q, K, V, _), (q, k, v, _), params, bm = problem(64, 128, "identity", 2)
    print("[case] paged forward", flush=True)
    pools = [t.reshape(1, 2, 64, 64).permute(1, 0, 2, 3).contiguous() for t in (k, v)]
    table = torch.tensor([[0, 1]], dtype=torch.int32, device=DEV)
    phys, phys_full = torch.empty_like(bm.kv_indices), torch.empty_like(bm.full_kv_indices)
    fa.flexattn_paged_convert_blockmask(bm.kv_num_blocks, bm.kv_indices, table, phys)
    fa.flexattn_paged_convert_blockmask(bm.full_kv_num_blocks, bm.full_kv_indices, table, phys_full)
    O, LSE = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device=DEV), torch.full(q.shape[:3], float("nan"), device=DEV)
    fa.flexattn_paged_forward(q, *pools, fa.SCORE_IDENTITY, fa.MASK_CAUSAL, params, bm, phys, phys_full, 0.125, O, LSE)
    torch.cuda.synchronize()
    hp.check_output(O[:, :1], LSE[:, :1], *fo.flex_attention(Q, K, V, fo.Identity(), fo.no_mask, 0.125))
    assert torch.equal(O, O[:, :1].expand_as(O)) and torch.equal(LSE, LSE[:, :1].expand_as(LSE))


def test_dq_and_captured_sums():
    """Rows long enough for four waves to share them."""
    import paper_2412_05496_amd as fa
    n, D = 800, 64
    (Q, K, V, dO), (q, k, v, do), params, bm = problem(D, n, "alibi", 3)
    score = fo.Alibi(torch.tensor([-0.01], dtype=torch.float64))
    off = torch.tensor([n - 1], dtype=torch.int32)
    score, mask = fo.QOffset(score, off), fo.with_q_offset(fo.causal_mask, off)
    ref = fo.flex_attention_backward(Q, K, V, dO, score, mask, 0.125)[0]
    O_ref, LSE_ref = fo.flex_attention(Q, K, V, score, mask, 0.125)
    print("[case] dQ, captured", flush=True)
    O, LSE = O_ref.to(torch.bfloat16).to(DEV).expand_as(q), LSE_ref.float().to(DEV).expand(1, HEADS, 1).contiguous()
    head = (fa.SCORE_ALIBI, fa.MASK_CAUSAL, params, bm, 0.125)
    dQ = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device=DEV)
    ws = torch.empty(fa.flexattn_backward_workspace_bytes(q, k), dtype=torch.uint8, device=DEV)
    fa.flexattn_backward_stages(q, k, v, O, do, LSE, *head, dQ, None, None, ws, 1 | 4)
    torch.cuda.synchronize()
    hp.check_grad("dQ", dQ[:, :1], ref)
    assert torch.equal(dQ, dQ[:, :1].expand_as(dQ))
    d_alibi = torch.full((HEADS,), float("nan"), device=DEV)
    fa.flexattn_backward_captured(q, k, v, O, do, LSE, *head, d_alibi, None)
    torch.cuda.synchronize()
    assert torch.isfinite(d_alibi[0]) and torch.equal(d_alibi, d_alibi[:1].expand_as(d_alibi))
