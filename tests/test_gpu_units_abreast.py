"""Heads whose rows (columns) of blocks take turns in a launch: whole sets, a last set with what is left over, heads beyond a multiple of eight.
The heads have the same inputs, so that a piece that is left out or done for another head shows up as a head unlike the first."""
import pytest
import torch

from oracle import flex_oracle as fo
from tests import helpers as hp

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("heads,S,D,Bq,doc", [
    (75, 150, 64, 128, 0),          # one set of nine, three heads over
    (136, 200, 64, 128, 0),         # sets of eight and nine (rows), of four and five (columns)
    (139, 130, 64, 64, 0),
    (72, 300, 128, 128, 0),
    (48, 700, 128, 64, 0),          # sets of six (rows)
    (40, 1000, 64, 128, 700),       # documents whose longest row is long, in halves and whole rows
    (136, 500, 64, 128, 30),        # and short: head by head
    (67, 400, 128, 128, 350),
    (44, 700, 128, 128, 60),        # short ones in rows of 128 queries, by heads that would take turns with dS in memory as well
])
def test_every_head_is_the_first(heads, S, D, Bq, doc):
    import paper_2412_05496_amd as fa
    print("[case]", heads, S, D, Bq, doc, flush=True)
    gen = torch.Generator().manual_seed(heads + S)
    Q, K, V, dO = (torch.randn(1, 1, S, D, generator=gen).to(torch.bfloat16) for _ in range(4))
    params, mask, mask_id = fa.ModParams(), fo.causal_mask, fa.MASK_CAUSAL
    if doc:
        ids = (torch.arange(S) // doc).to(torch.int32).view(1, S)
        params.doc_ids = ids.to(DEV)
        mask, mask_id = fo.and_mask(fo.document_mask(ids), fo.causal_mask), fa.MASK_DOCUMENT_CAUSAL
    scale = D ** -0.5
    bm = fa.alloc_blockmask(1, 1, S, S, Bq, 64, device=DEV)
    fa.flexattn_blockmask_build(mask_id, params, bm)
    q, k, v, do = (t.to(DEV).expand(1, heads, S, D) for t in (Q, K, V, dO))
    O, dQ, dK, dV = (torch.full((1, heads, S, D), float("nan"), dtype=torch.bfloat16, device=DEV) for _ in range(4))
    LSE = torch.full((1, heads, S), float("nan"), device=DEV)
    head = (fa.SCORE_IDENTITY, mask_id, params, bm, scale)
    fa.flexattn_forward(q, k, v, *head, O, LSE)
    fa.flexattn_backward(q, k, v, O, do, LSE, *head, dQ, dK, dV)
    torch.cuda.synchronize()
    hp.check_output(O[:, :1], LSE[:, :1], *fo.flex_attention(Q, K, V, fo.Identity(), mask, scale))
    for name, got, ref in zip(("dQ", "dK", "dV"), (dQ, dK, dV), fo.flex_attention_backward(Q, K, V, dO, fo.Identity(), mask, scale)):
        hp.check_grad(name, got[:, :1], ref)
    for got in (O, LSE, dQ, dK, dV):
        assert torch.equal(got, got[:, :1].expand_as(got))
    # dS through memory, whose dQ kernel goes by the same order
    n_blocks = hp.nonempty_blocks(bm)
    ws = hp.dirty_stored_workspace(q, k, bm, n_blocks)
    dQ.fill_(float("nan"))
    for stages in (1, 2, 4):
        fa.flexattn_backward_stored(q, k, v, O, do, LSE, *head, dQ, dK, dV, n_blocks, ws, stages)
    torch.cuda.synchronize()
    hp.check_grad("dQ*", dQ[:, :1], fo.flex_attention_backward(Q, K, V, dO, fo.Identity(), mask, scale)[0])
    assert torch.equal(dQ, dQ[:, :1].expand_as(dQ))
