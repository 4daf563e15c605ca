"""dK/dV, in the kernels whose waves exchange P and dS, of columns of blocks that list steps of 64 queries which the indices alone hide from the 64 keys: at a diagonal, at
a window's far edge, behind the last query, in columns without a visible one, and more of them than one entry of the walk counts.
Gradients against the oracle, recomputed and with dS in memory (whose hidden steps must read as zeros)."""
import pytest
import torch

from oracle import flex_oracle as fo
from tests import helpers as hp

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def gradients(mask_id, mask_mod, S, Bq, Bk, params, everything=False, Hq=2, Hkv=1, B=0, q_len=None, capped=False):
    """everything: all blocks are listed as PARTIAL, whatever the mask hides of them.  The entries of the batch have the same inputs: every one is compared."""
    import paper_2412_05496_amd as fa
    D, q_len = 64 if capped else 128, q_len or S
    parts = B > 0               # (the groups' heads are divided)
    B = B or 60000 // S + 1     # (more than 768 workgroups: all that run at once look for no steps to leave out)
    score_id, score = fa.SCORE_IDENTITY, fo.Identity()
    if capped:                  # (at D = 64 a bias and a soft-cap take that kernel)
        bias = torch.tensor([-0.03, 0.01])[:Hq]
        params.alibi_bias, params.softcap = bias.to(DEV), 30.0
        score_id, score = fa.SCORE_ALIBI | fa.SCORE_SOFTCAP, fo.Compose(fo.Alibi(bias), fo.Softcap(30.0))
    if mask_id == fa.MASK_SWA_CAUSAL_OR_PREFIX:         # (compiled with a relative bias)
        table = 0.3 * torch.randn(Hq, 90, generator=torch.Generator().manual_seed(3))
        params.rel_bias = table.to(DEV)
        score_id, score = fa.SCORE_REL_BIAS, fo.RelBias(table.double())
    g = torch.Generator().manual_seed(S + Bq + Bk)
    Q, dO = (torch.randn(1, Hq, q_len, D, generator=g).to(torch.bfloat16) for _ in range(2))
    K, V = (torch.randn(1, Hkv, S, D, generator=g).to(torch.bfloat16) for _ in range(2))
    refs = fo.flex_attention_backward(*(t.float() for t in (Q, K, V, dO)), score, mask_mod, D ** -0.5)
    bm = fa.alloc_blockmask(1, 1, q_len, S, Bq, Bk, device=torch.device(DEV))
    fa.flexattn_blockmask_build(mask_id, params, bm)
    if everything:
        NR, NC = (q_len + Bq - 1) // Bq, (S + Bk - 1) // Bk
        for num, idx, full, n in ((bm.kv_num_blocks, bm.kv_indices, bm.full_kv_num_blocks, NC), (bm.q_num_blocks, bm.q_indices, bm.full_q_num_blocks, NR)):
            num.fill_(n)
            full.zero_()
            idx.copy_(torch.arange(n, dtype=torch.int32).expand(idx.shape))
        bm.stats[0], bm.stats[1] = NR * NC, 0
    Q, K, V, dO = (t.to(DEV).expand(B, -1, -1, -1) for t in (Q, K, V, dO))
    unwritten = lambda t: torch.full(t.shape, float("nan"), dtype=t.dtype, device=DEV)
    O, LSE = unwritten(Q), torch.full((B, Hq, q_len), float("nan"), device=DEV)
    head = (score_id, mask_id, params, bm, D ** -0.5)
    fa.flexattn_forward(Q, K, V, *head, O, LSE)
    n = hp.nonempty_blocks(bm)
    for stored in (False, True):
        dQ, Vs, _ = hp.dq_and_v_in_one_storage(Q, V)
        got = [dQ, unwritten(K), unwritten(V)]
        if stored:
            ws = hp.dirty_stored_workspace(Q, K, bm, n)
            fa.flexattn_backward_stored(Q, K, Vs, O, dO, LSE, *head, *got, n, ws)
            assert hp.ds_written(ws, bm, n)
        else:
            got[0] = unwritten(Q)
            ws = torch.full((max(fa.flexattn_backward_workspace_bytes(Q, K), 1),), 0xFF, dtype=torch.uint8, device=DEV)
            fa.flexattn_backward(Q, K, V, O, dO, LSE, *head, *got, ws)
        torch.cuda.synchronize()
        room = hp.room_for_parts(Q, K)
        assert bool((ws[ws.numel() - room:] != 0xFF).any()) == parts
        for name, t, ref in zip(("dQ", "dK", "dV"), got, refs):
            hp.check_grad(name, t[:1], ref)
            assert torch.equal(t, t[:1].expand_as(t)), name


MASKS = {"causal": lambda fa, w: (fa.MASK_CAUSAL, fo.causal_mask, fa.ModParams()),
         "capped": lambda fa, w: (fa.MASK_CAUSAL, fo.causal_mask, fa.ModParams()),
         "none": lambda fa, w: (fa.MASK_NONE, fo.no_mask, fa.ModParams()),
         "window": lambda fa, w: (fa.MASK_SWA_CAUSAL, fo.and_mask(fo.causal_mask, fo.sliding_window_mask(w)), fa.ModParams(window=w)),
         "biased": lambda fa, w: (fa.MASK_SWA_CAUSAL_OR_PREFIX, fo.or_mask(fo.and_mask(fo.causal_mask, fo.sliding_window_mask(w)), fo.prefix_mask(40)),
                                  fa.ModParams(window=w, prefix_len=40)),
         "prefix": lambda fa, w: (fa.MASK_PREFIX_LM, fo.or_mask(fo.causal_mask, fo.prefix_mask(w)), fa.ModParams(prefix_len=w))}


@pytest.mark.parametrize("Bq,Bk", [(128, 64), (64, 128), (128, 128), (64, 64)])
@pytest.mark.parametrize("mask,S,w", [("capped", 300, 0), ("capped", 1100, 0), ("causal", 300, 0), ("causal", 1100, 0), ("none", 777, 0), ("window", 1000, 195),
                                      ("window", 830, 31), ("prefix", 700, 130), ("biased", 300, 100),
                                      ("biased", 1000, 195)])
def test_hidden_steps(mask, S, w, Bq, Bk):
    import paper_2412_05496_amd as fa
    mask_id, mask_mod, params = MASKS[mask](fa, w)
    print(f"[case] {mask} S={S} blocks {Bq}x{Bk}", flush=True)
    gradients(mask_id, mask_mod, S, Bq, Bk, params, capped=mask == "capped")


@pytest.mark.parametrize("mask,S,w", [("capped", 2500, 0), ("causal", 2500, 0), ("window", 2500, 100), ("causal", 5000, 0), ("window", 4200, 70), ("biased", 2500, 100)])
def test_lists_full_of_hidden_blocks(mask, S, w):
    """Up to 39, 39, 38, 78, 65 and 38 hidden steps in a column's list: fewer than an entry counts and more, fewer than 64 in a row and more."""
    import paper_2412_05496_amd as fa
    mask_id, mask_mod, params = MASKS[mask](fa, w)
    print(f"[case] {mask} S={S}", flush=True)
    gradients(mask_id, mask_mod, S, 64 if S < 3000 else 128, 128 if S < 3000 else 64, params, everything=True, Hq=1, capped=mask == "capped")


def test_columns_without_a_visible_step():
    import paper_2412_05496_amd as fa
    mask_id, mask_mod, params = MASKS["causal"](fa, 0)
    gradients(mask_id, mask_mod, 700, 128, 64, params, everything=True, q_len=200)


@pytest.mark.parametrize("mask,S,w,Bq,Bk,Hq,Hkv,B", [
    ("causal", 1100, 0, 128, 128, 16, 2, 4), ("window", 1600, 1400, 128, 128, 8, 1, 6), ("prefix", 1100, 130, 64, 128, 16, 2, 4), ("causal", 2100, 0, 128, 64, 8, 4, 2)])
def test_hidden_steps_of_divided_groups(mask, S, w, Bq, Bk, Hq, Hkv, B):
    """Of 513 to 768 workgroups: the heads of a group are divided, and each part leaves its hidden steps out."""
    import paper_2412_05496_amd as fa
    mask_id, mask_mod, params = MASKS[mask](fa, w)
    print(f"[case] {mask} S={S} blocks {Bq}x{Bk} heads {B} x {Hq} / {Hkv}", flush=True)
    gradients(mask_id, mask_mod, S, Bq, Bk, params, Hq=Hq, Hkv=Hkv, B=B)
