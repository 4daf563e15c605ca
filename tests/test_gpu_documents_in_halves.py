"""Packed documents with rows of blocks of 128 in launches that take the longest third of the rows in halves of 64 and the others
whole, or, where the longest row of a sequence is short, all whole.  Both in one batch; rows of blocks that are no multiple of three, a
last half without a row; one plane for all heads and a plane per head, grouped heads, no work order (the longest rows are then not the
first).  Against the oracle at the tolerances of tests/helpers.py, copies bit for bit the same."""
import pytest
import torch

import flex_workloads as wlm
from oracle import flex_oracle as fo
from tests import helpers as hp

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def packed(S, lo, hi, seed):
    gen = torch.Generator().manual_seed(seed)
    out = []
    while len(out) < S:
        out += [len(out)] * int(torch.randint(lo, hi + 1, (1,), generator=gen))
    return torch.tensor(out[:S], dtype=torch.int32)


@pytest.mark.parametrize("score,D,S,Bk,heads,copies", [
    ("identity", 64, 2100, 64, (1, 1), 12), ("alibi", 64, 2111, 64, (4, 2), 5), ("rel_bias_softcap", 64, 2304, 128, (2, 1), 6),
    ("identity", 64, 2500, 128, (2, 2), 9), ("identity", 128, 2060, 64, (2, 1), 3), ("alibi", 128, 2240, 128, (1, 1), 8), ("alibi", 128, 2049, 64, (3, 1), 2)])
@pytest.mark.parametrize("planes", ["shared", "per_head", "no_order"])
def test_long_and_short_documents(score, D, S, Bk, heads, copies, planes):
    import paper_2412_05496_amd as fa
    Hq, Hkv = heads
    wl = wlm.CFG1.scaled(name="mixed", B=1, Hq=Hq, Hkv=Hkv, S=S, D=D, Bq=128, Bk=Bk, mask="doc_causal", score=score, softcap=20.0, rel_len=50,
                         doc_len_min=100, doc_len_max=700, seed=6100 + S)
    inp = wlm.make_train_inputs(wl, with_dO=True)
    mask_id, score_id, params, _ = hp.library_mods(wl, inp, DEV)
    # sequences with long rows, short ones, and rows of one document's length on both sides of what is short
    docs = [packed(S, *d) for d in ((300, 1500, S), (16, 100, 1), (200, 500, 2), (1, 5, 3), (380, 420, 4))]
    params.doc_ids = torch.stack(docs).repeat(copies, 1).contiguous().to(DEV)
    B = len(docs) * copies
    bm = fa.alloc_blockmask(B, Hq if planes == "per_head" else 1, S, S, 128, Bk, device=DEV, work_order=planes != "no_order")
    fa.flexattn_blockmask_build(mask_id, params, bm)
    Q, K, V, dO = (t.to(DEV).expand(B, -1, -1, -1) for t in (inp.Q, inp.K, inp.V, inp.dO))
    O, LSE = torch.full(Q.shape, float("nan"), dtype=torch.bfloat16, device=DEV), torch.full(Q.shape[:3], float("nan"), device=DEV)
    head = (score_id, mask_id, params, bm, inp.scale)
    print(f"[case] {score} D={D} S={S} Bk={Bk} heads={Hq}/{Hkv} {planes}", flush=True)
    fa.flexattn_forward(Q, K, V, *head, O, LSE)
    grads = [torch.full(t.shape, float("nan"), dtype=torch.bfloat16, device=DEV) for t in (Q, K, V)]
    fa.flexattn_backward(Q, K, V, O, dO, LSE, *head, *grads)
    torch.cuda.synchronize()
    n = len(docs)
    for t in (O, LSE, *grads):
        assert torch.equal(t, t[:n].repeat(copies, *[1] * (t.dim() - 1)))
    score_mod, _ = hp.oracle_mods(wl, inp)
    for i, ids in enumerate(docs):
        mask = fo.and_mask(fo.document_mask(ids.view(1, -1)), fo.causal_mask)
        hp.check_output(O[i:i + 1], LSE[i:i + 1], *fo.flex_attention(inp.Q, inp.K, inp.V, score_mod, mask, inp.scale))
        for name, got, ref in zip(("dQ", "dK", "dV"), grads, fo.flex_attention_backward(inp.Q, inp.K, inp.V, inp.dO, score_mod, mask, inp.scale)):
            hp.check_grad(name, got[i:i + 1], ref)
