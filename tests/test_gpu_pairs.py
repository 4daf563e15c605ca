"""Forward, dQ and captured sums where a workgroup is two slices of 32 rows times the two key halves of every tile: rows of
blocks of 64, and the halves of 128-row blocks of uneven rows.  Ragged ends (a slice or a half without a row), both sides of
the lines that choose the form, rows that only one of the two waves sees keys of, grouped heads.  Against the oracle at the
tolerances of tests/helpers.py."""
import pytest
import torch

import flex_workloads as wlm
from oracle import flex_oracle as fo
from tests import helpers as hp

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def check(wl, copies, captured=False):
    import paper_2412_05496_amd as fa
    dev = torch.device(DEV)
    inp = wlm.make_train_inputs(wl, with_dO=True)
    score_mod, mask_mod = hp.oracle_mods(wl, inp)
    mask_id, score_id, params, _ = hp.library_mods(wl, inp, dev)
    print(f"[case] {wl.mask} {wl.score} D={wl.D} S={wl.S} Bq={wl.Bq} heads={wl.Hq}/{wl.Hkv} copies={copies}", flush=True)
    O_ref, LSE_ref = fo.flex_attention(inp.Q, inp.K, inp.V, score_mod, mask_mod, inp.scale)
    refs = fo.flex_attention_backward(inp.Q, inp.K, inp.V, inp.dO, score_mod, mask_mod, inp.scale)
    bm = fa.alloc_blockmask(1, 1, wl.S, wl.S, wl.Bq, wl.Bk, device=dev)
    if params.doc_ids is not None:
        params.doc_ids = params.doc_ids[:1].expand(copies, -1).contiguous()
    fa.flexattn_blockmask_build(mask_id, params, bm)
    Q, K, V, dO = (t.to(dev).expand(copies, -1, -1, -1) for t in (inp.Q, inp.K, inp.V, inp.dO))
    O, LSE = torch.full(Q.shape, float("nan"), dtype=torch.bfloat16, device=dev), torch.full(Q.shape[:3], float("nan"), device=dev)
    head = (score_id, mask_id, params, bm, inp.scale)
    fa.flexattn_forward(Q, K, V, *head, O, LSE)
    grads = [torch.full(t.shape, float("nan"), dtype=torch.bfloat16, device=dev) for t in (Q, K, V)]
    fa.flexattn_backward(Q, K, V, O, dO, LSE, *head, *grads)
    torch.cuda.synchronize()
    hp.check_output(O[:1], LSE[:1], O_ref, LSE_ref)
    assert torch.equal(O, O[:1].expand_as(O)) and torch.equal(LSE, LSE[:1].expand_as(LSE))
    for name, got, ref in zip(("dQ", "dK", "dV"), grads, refs):
        hp.check_grad(name, got[:1], ref)
        assert torch.equal(got, got[:1].expand_as(got)), name
    if captured:
        # the same dS as with rows of blocks of 128, added up in another order: fp32 sums of chains of up to S terms
        bm128 = fa.alloc_blockmask(1, 1, wl.S, wl.S, 128, wl.Bk, device=dev)
        fa.flexattn_blockmask_build(mask_id, params, bm128)
        sums = [torch.full((wl.Hq,), float("nan"), device=dev) for _ in range(2)]
        for blocks, d_alibi in zip((bm, bm128), sums):
            fa.flexattn_backward_captured(Q[:1], K[:1], V[:1], O[:1], dO[:1], LSE[:1], score_id, mask_id, params, blocks, inp.scale, d_alibi, None)
        torch.cuda.synchronize()
        bound = wl.S * 2.0 ** -24 * size_of_terms(inp, wl, score_mod, mask_mod)
        print("  captured", sums[0].tolist(), sums[1].tolist(), bound.tolist(), flush=True)
        assert ((sums[0] - sums[1]).double().cpu().abs() <= bound).all()


def size_of_terms(inp, wl, score_mod, mask_mod):
    """Per head, the sum of |dS (q - kv)|, in 64 bits."""
    pos = torch.arange(wl.S)
    q, kv = pos.view(-1, 1), pos.view(1, -1)
    out = []
    for h in range(wl.Hq):
        Qh, Kh, Vh, dOh = (t[0, i].double() for t, i in ((inp.Q, h), (inp.K, h * wl.Hkv // wl.Hq), (inp.V, h * wl.Hkv // wl.Hq), (inp.dO, h)))
        s = Qh @ Kh.T * inp.scale - inp.slopes[h].double() * (q - kv)
        P = torch.softmax(s.masked_fill(~mask_mod(0, h, q, kv), float("-inf")), dim=-1)
        dP = dOh @ Vh.T
        out.append((P * (dP - (P * dP).sum(-1, keepdim=True)) * (q - kv)).abs().sum())
    return torch.stack(out)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("mask,score,S,Bk,heads,copies", [
    ("causal", "identity", 449, 64, (2, 1), 130), ("causal", "alibi", 780, 128, (2, 2), 40), ("none", "identity", 769, 64, (1, 1), 130),
    ("swa_causal", "softcap", 930, 64, (2, 1), 60), ("doc_causal", "alibi", 850, 64, (2, 2), 40), ("prefix_lm", "identity", 800, 128, (1, 1), 100),
    ("causal", "identity", 33, 64, (1, 1), 1100), ("swa_causal_or_prefix", "rel_bias", 801, 64, (2, 1), 60)])
def test_rows_of_blocks_of_64(mask, score, S, Bk, heads, copies, D):
    wl = wlm.CFG1.scaled(name="pairs64", B=1, Hq=heads[0], Hkv=heads[1], S=S, D=D, Bq=64, Bk=Bk, mask=mask, score=score, window=700,
                         prefix_len=300, softcap=20.0, rel_len=50, doc_len_min=100, doc_len_max=400, seed=5100 + S)
    check(wl, copies, captured=score == "alibi")


@pytest.mark.parametrize("mask,score,D,S,Bk,copies", [
    ("causal", "identity", 64, 2100, 64, 40), ("causal", "softcap", 64, 2176, 128, 56), ("doc_causal", "alibi", 64, 2111, 64, 110),
    ("prefix_lm", "identity", 64, 2050, 64, 45), ("causal", "identity", 128, 2100, 64, 24), ("doc_causal", "alibi", 128, 2060, 128, 40),
    ("causal", "alibi", 128, 2048, 64, 30), ("causal", "identity", 64, 2047, 64, 60),
    ("none", "identity", 64, 1100, 64, 40), ("none", "identity", 64, 1024, 128, 64), ("causal", "softcap", 64, 1025, 64, 50)])
def test_halves_of_128_row_blocks(mask, score, D, S, Bk, copies):
    wl = wlm.CFG1.scaled(name="pairs128", B=1, Hq=1, Hkv=1, S=S, D=D, Bq=128, Bk=Bk, mask=mask, score=score, window=700,
                         prefix_len=300, softcap=20.0, doc_len_min=100, doc_len_max=700, seed=5200 + S)
    check(wl, copies)


@pytest.mark.parametrize("mask,score,S,Hq,Hkv,Bk,B", [
    ("causal", "softcap", 4100, 2, 1, 64, 8), ("swa_causal", "softcap", 4480, 4, 2, 64, 4),    # two heads to a workgroup
    ("causal", "softcap", 4100, 3, 3, 64, 11), ("none", "identity", 4001, 3, 1, 128, 11),       # two rows of blocks (33, 32 of them)
    ("prefix_lm", "identity", 4160, 1, 1, 64, 32)])
def test_stored_dq_that_shares_k_tiles(mask, score, S, Hq, Hkv, Bk, B):
    """dQ through memory is the recomputed one up to the order of its fp32 sums: one bf16 rounding of each, 2^-8 of the larger
    values.  The workspace starts as NaN patterns, dS of blocks that a row does not list is not read."""
    import paper_2412_05496_amd as fa
    dev = torch.device(DEV)
    gen = torch.Generator(device=dev).manual_seed(S + Hq)
    Q, dO = (torch.randn(B, Hq, S, 128, generator=gen, device=dev).to(torch.bfloat16) for _ in range(2))
    K, V = (torch.randn(B, Hkv, S, 128, generator=gen, device=dev).to(torch.bfloat16) for _ in range(2))
    params = fa.ModParams(softcap=30.0, window=4200, prefix_len=500)
    mask_id = {"causal": fa.MASK_CAUSAL, "none": fa.MASK_NONE, "swa_causal": fa.MASK_SWA_CAUSAL, "prefix_lm": fa.MASK_PREFIX_LM}[mask]
    score_id = fa.SCORE_SOFTCAP if score == "softcap" else fa.SCORE_IDENTITY
    print(f"[case] {mask} {score} S={S} heads={Hq}/{Hkv} Bk={Bk} B={B}", flush=True)
    bm = fa.alloc_blockmask(1, 1, S, S, 128, Bk, device=dev)
    fa.flexattn_blockmask_build(mask_id, params, bm)
    O, LSE = torch.empty_like(Q), torch.empty(B, Hq, S, dtype=torch.float32, device=dev)
    head = (score_id, mask_id, params, bm, 128 ** -0.5)
    fa.flexattn_forward(Q, K, V, *head, O, LSE)
    want = [torch.empty_like(t) for t in (Q, K, V)]
    fa.flexattn_backward(Q, K, V, O, dO, LSE, *head, *want)
    n = hp.nonempty_blocks(bm)
    ws = hp.dirty_stored_workspace(Q, K, bm, n)
    got = [torch.full_like(t, float("nan")) for t in (Q, K, V)]
    fa.flexattn_backward_stored(Q, K, V, O, dO, LSE, *head, *got, n, ws)
    torch.cuda.synchronize()
    assert hp.ds_written(ws, bm, n)
    assert torch.equal(got[1], want[1]) and torch.equal(got[2], want[2])
    err = (got[0].float() - want[0].float()).abs()
    assert torch.isfinite(got[0].float()).all() and err.max() <= 2 ** -7 * want[0].float().abs().max()
    assert err.mean() <= 2 ** -9 * want[0].float().abs().mean()
