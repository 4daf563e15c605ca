"""Launches that leave the chip idle split the keys (forward, dQ) or query rows (dK/dV) of a few rows (keys) among the waves of
a workgroup; larger ones give every wave rows (keys) of its own.  The same problem through both: alone, and as many copies
in one batch, each against the oracle, the copies bit for bit the same."""
import pytest
import torch

import flex_workloads as wlm
from oracle import flex_oracle as fo
from tests import helpers as hp

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

MODS = [("none", "identity", {}), ("causal", "identity", {}), ("causal", "alibi", {}), ("causal", "softcap", {"softcap": 30.0}),
        ("causal", "softcap", {"softcap": 60.0}), ("swa_causal", "identity", {"window": 90}), ("prefix_lm", "identity", {"prefix_len": 70}),
        ("doc_causal", "identity", {"doc_len_min": 1, "doc_len_max": 9}), ("doc_causal", "alibi", {"doc_len_min": 30, "doc_len_max": 200}),
        ("swa_causal_or_prefix", "rel_bias", {"window": 100, "prefix_len": 40, "rel_len": 64}), ("swa_causal", "softcap", {"window": 64, "softcap": 20.0}),
        ("causal", "alibi_softcap", {"softcap": 30.0}),
        ("doc_causal", "rel_bias_softcap", {"rel_len": 33, "doc_len_min": 20, "doc_len_max": 150, "softcap": 50.0})]
COPIES = 48         # of two heads of 14 slices of 32 rows: beyond every line at this length


def run(mask_id, score_id, params, Bm, t, scale, Bq, Bk, stored):
    import paper_2412_05496_amd as fa
    Q, K, V, dO = t
    bm = fa.alloc_blockmask(Bm, 1, Q.shape[2], K.shape[2], Bq, Bk, device=DEV)
    fa.flexattn_blockmask_build(mask_id, params, bm)
    nan = lambda x: torch.full_like(x, float("nan"))
    O, LSE = nan(Q), torch.full(Q.shape[:3], float("nan"), dtype=torch.float32, device=DEV)
    fa.flexattn_forward(Q, K, V, score_id, mask_id, params, bm, scale, O, LSE)
    dQ, dK, dV = nan(Q), nan(K), nan(V)
    args = (Q, K, V, O, dO, LSE, score_id, mask_id, params, bm, scale, dQ, dK, dV)
    if stored:
        fa.flexattn_backward_stored(*args, hp.nonempty_blocks(bm))
    else:
        fa.flexattn_backward(*args)
    torch.cuda.synchronize()
    return O, LSE, dQ, dK, dV


@pytest.mark.parametrize("D,S,Bq,Bk", [(64, 419, 128, 64), (128, 419, 128, 64), (64, 420, 64, 128), (128, 417, 64, 128)])
@pytest.mark.parametrize("mask,score,over", MODS, ids=[f"{m[0]}-{m[1]}-{i}" for i, m in enumerate(MODS)])
def test_alone_and_in_a_batch(mask, score, over, D, S, Bq, Bk):
    wl = wlm.CFG1.scaled(name="few_many", B=1, Hq=2, Hkv=1, S=S, D=D, Bq=Bq, Bk=Bk, mask=mask, score=score, seed=9100 + S, backward=True, **over)
    inp = wlm.make_train_inputs(wl, with_dO=True)
    score_mod, mask_mod = hp.oracle_mods(wl, inp)
    O_ref, LSE_ref = fo.flex_attention(inp.Q, inp.K, inp.V, score_mod, mask_mod, inp.scale)
    ref = fo.flex_attention_backward(inp.Q, inp.K, inp.V, inp.dO, score_mod, mask_mod, inp.scale)
    mask_id, score_id, params, _ = hp.library_mods(wl, inp, DEV)
    one = [x.to(DEV) for x in (inp.Q, inp.K, inp.V, inp.dO)]
    many = [x.repeat(COPIES, 1, 1, 1) for x in one]
    docs = params.doc_ids
    for copies, tensors in ((1, one), (COPIES, many)):
        if docs is not None:
            params.doc_ids = docs.reshape(1, -1).repeat(copies, 1)
        for stored in (False, True):
            out = run(mask_id, score_id, params, copies if docs is not None else 1, tensors, inp.scale, Bq, Bk, stored)
            for x in out:
                assert torch.equal(x, x[:1].expand_as(x))
            hp.check_output(out[0][:1], out[1][:1], O_ref, LSE_ref)
            for name, got, want in zip(("dQ", "dK", "dV"), out[2:], ref):
                hp.check_grad(name, got[:1], want)


@pytest.mark.parametrize("W,H,K,layout,tile,D", [(28, 20, 7, "row_major", 0, 64), (32, 16, 9, "tiled", 8, 128), (16, 16, 5, "morton", 0, 64)])
def test_canvas_alone_and_in_a_batch(W, H, K, layout, tile, D):
    import paper_2412_05496_amd as fa
    S = W * H
    wl = wlm.CFG1.scaled(name="few_many_canvas", B=1, Hq=2, Hkv=2, S=S, D=D, Bq=128, Bk=64, mask="none", score="identity", seed=9200 + S, backward=True)
    inp = wlm.make_train_inputs(wl, with_dO=True)
    mask_mod = fo.neighborhood_mask(W, H, K, layout, tile)
    O_ref, LSE_ref = fo.flex_attention(inp.Q, inp.K, inp.V, fo.Identity(), mask_mod, inp.scale)
    ref = fo.flex_attention_backward(inp.Q, inp.K, inp.V, inp.dO, fo.Identity(), mask_mod, inp.scale)
    params = fa.ModParams(na_width=W, na_height=H, na_kernel=K, na_layout={"row_major": 0, "tiled": 1, "morton": 2}[layout], na_tile=tile)
    one = [x.to(DEV) for x in (inp.Q, inp.K, inp.V, inp.dO)]
    for copies in (1, 1 + 1100 // (S // 16)):
        for stored in (False, True):
            out = run(fa.MASK_NEIGHBORHOOD, fa.SCORE_IDENTITY, params, 1, [x.repeat(copies, 1, 1, 1) for x in one], inp.scale, 128, 64, stored)
            for x in out:
                assert torch.equal(x, x[:1].expand_as(x))
            hp.check_output(out[0][:1], out[1][:1], O_ref, LSE_ref)
            for name, got, want in zip(("dQ", "dK", "dV"), out[2:], ref):
                hp.check_grad(name, got[:1], want)


@pytest.mark.parametrize("D,page,copies", [(64, 64, 1), (64, 128, 24), (128, 64, 1), (128, 128, 16)])
def test_paged_alone_and_in_a_batch(D, page, copies):
    import paper_2412_05496_amd as fa
    kv_lens, q_len = [700, 97, 1000, 512], 97
    wl = wlm.CFG5.scaled(name="few_many_paged", B=4, Hq=4, Hkv=2, D=D, page_size=page, max_pages=1024 // page, mask="causal", score="identity",
                         S=q_len, Bq=128, Bk=page, seed=9300 + page)
    inp = wlm.make_prefill_inputs(wl, kv_lens, q_len, slack_pages=2)
    O_ref, LSE_ref = fo.paged_attention(inp.Q, inp.K_pool, inp.V_pool, inp.page_table, inp.kv_lens, inp.q_offsets, fo.Identity(),
                                        fo.causal_mask, inp.scale)
    rep = lambda t: t.to(DEV).repeat(copies, *([1] * (t.dim() - 1)))
    Q, table = rep(inp.Q), rep(inp.page_table)
    params = fa.ModParams(q_offsets=rep(inp.q_offsets))
    bm = fa.alloc_blockmask(4 * copies, 1, q_len, 1024, 128, page, device=DEV)
    fa.flexattn_blockmask_build(fa.MASK_CAUSAL, params, bm)
    phys, phys_full = torch.zeros_like(bm.kv_indices), torch.zeros_like(bm.full_kv_indices)
    fa.flexattn_paged_convert_blockmask(bm.kv_num_blocks, bm.kv_indices, table, phys)
    fa.flexattn_paged_convert_blockmask(bm.full_kv_num_blocks, bm.full_kv_indices, table, phys_full)
    O, LSE = torch.full_like(Q, float("nan")), torch.full(Q.shape[:3], float("nan"), dtype=torch.float32, device=DEV)
    fa.flexattn_paged_forward(Q, inp.K_pool.to(DEV), inp.V_pool.to(DEV), fa.SCORE_IDENTITY, fa.MASK_CAUSAL, params, bm, phys, phys_full, inp.scale, O, LSE)
    torch.cuda.synchronize()
    hp.check_output(O[:4], LSE[:4], O_ref, LSE_ref)
    assert torch.equal(O, O[:4].repeat(copies, 1, 1, 1)) and torch.equal(LSE, LSE[:4].repeat(copies, 1, 1))


@pytest.mark.parametrize("copies", [1, COPIES])
@pytest.mark.parametrize("over", ["Q", "dO", "O"])
def test_dq_written_over_a_tensor_of_its_shape(over, copies):
    """dQ may take the memory of Q, dO or O: nothing reads a row of theirs after its dQ has been written."""
    import paper_2412_05496_amd as fa
    wl = wlm.CFG1.scaled(name="dq_over", B=copies, Hq=2, Hkv=1, S=419, D=64, mask="causal", score="identity", seed=9300)
    inp = wlm.make_train_inputs(wl, with_dO=True)
    mask_id, score_id, params, _ = hp.library_mods(wl, inp, DEV)
    t = [x.to(DEV) for x in (inp.Q, inp.K, inp.V, inp.dO)]
    bm = fa.alloc_blockmask(1, 1, wl.S, wl.S, wl.Bq, wl.Bk, device=DEV)
    fa.flexattn_blockmask_build(mask_id, params, bm)
    for stored in (False, True):
        O, LSE, *want = run(mask_id, score_id, params, 1, t, inp.scale, wl.Bq, wl.Bk, stored)
        Q, K, V, dO = (x.clone() for x in t)
        dQ, dK, dV = {"Q": Q, "dO": dO, "O": O}[over], torch.empty_like(K), torch.empty_like(V)
        args = (Q, K, V, O, dO, LSE, score_id, mask_id, params, bm, inp.scale, dQ, dK, dV)
        if stored:
            fa.flexattn_backward_stored(*args, hp.nonempty_blocks(bm))
        else:
            fa.flexattn_backward(*args)
        torch.cuda.synchronize()
        for got, ref in zip((dQ, dK, dV), want):
            assert torch.equal(got, ref)
