"""GPU parity where the per-lane bit masks and token tags of PARTIAL blocks can go wrong: document ids that
are not packed (many distinct ids in 32 tokens, negative and large ones), canvases of one row or one
column, windows as large as the canvas, and BlockMask lines longer than a workgroup takes at once.
BlockMasks bit for bit; O, LSE and gradients at the tolerances of tests/helpers.py."""
import pytest
import torch

import flex_workloads as wlm
from oracle import flex_oracle as fo
from tests import helpers as hp

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def scattered_ids(B, S, n_ids, seed):
    g = torch.Generator().manual_seed(seed)
    names = torch.tensor([-5, 0, 2 ** 31 - 1, -2 ** 31, 7] + list(range(100, 200)), dtype=torch.int64)[:n_ids]
    return names[torch.randint(0, n_ids, (B, S), generator=g)].to(torch.int32).contiguous()


@pytest.mark.parametrize("D,score,Bq,Bk,S,n_ids", [
    (64, "identity", 128, 64, 320, 40),      # up to 32 distinct ids in 32 tokens
    (64, "alibi", 64, 128, 257, 3),
    (128, "rel_bias_softcap", 128, 64, 200, 5),
    (128, "alibi", 128, 128, 129, 1),        # one document: the tags never hide anything
    (64, "identity", 128, 64, 300, 9),       # about as many ids as are matched by a ballot each
    (128, "identity", 128, 64, 333, 10),
    (128, "rel_bias_softcap", 64, 64, 200, 60),
])
def test_scattered_documents(D, score, Bq, Bk, S, n_ids):
    dev = torch.device(DEV)
    wl = wlm.CFG3.scaled(name="scattered", B=2, Hq=2, Hkv=1, S=S, D=D, Bq=Bq, Bk=Bk, score=score, softcap=20.0, rel_len=40,
                         doc_len_min=50, doc_len_max=90, seed=4100 + S)
    inp = wlm.make_train_inputs(wl, with_dO=True)
    inp.doc_ids = scattered_ids(2, S, n_ids, seed=S)
    score_mod, mask_mod = hp.oracle_mods(wl, inp)
    print(f"[case] scattered documents D={D} {score} S={S} ids={n_ids}", flush=True)
    O, LSE, bm, ids = hp.run_forward(wl, inp, dev)
    hp.assert_blockmask_equal(bm, fo.create_block_mask(mask_mod, 2, 1, S, S, Bq, Bk))
    hp.check_output(O, LSE, *fo.flex_attention(inp.Q, inp.K, inp.V, score_mod, mask_mod, inp.scale))
    ref = fo.flex_attention_backward(inp.Q, inp.K, inp.V, inp.dO, score_mod, mask_mod, inp.scale)
    for stored in (False, True):
        for name, got, r in zip(("dQ", "dK", "dV"), hp.run_backward(wl, inp, dev, O, LSE, bm, ids, stored=stored), ref):
            hp.check_grad(name, got, r)


@pytest.mark.parametrize("mask,score,S,Bq,Bk,Hkv", [
    ("causal", "identity", 65, 128, 64, 2), ("causal", "softcap", 160, 64, 128, 1), ("none", "identity", 33, 128, 64, 2),
    ("swa_causal", "identity", 330, 128, 128, 1), ("prefix_lm", "identity", 200, 128, 64, 2), ("causal", "alibi", 257, 64, 64, 1),
    ("swa_causal_or_prefix", "rel_bias", 290, 128, 64, 1), ("causal", "alibi_softcap", 190, 128, 64, 2)])
@pytest.mark.parametrize("extra_keys", [0, 100])
def test_blocks_hidden_from_a_wave(mask, score, S, Bq, Bk, Hkv, extra_keys):
    """D = 64 gradients where 32 x 32 blocks of PARTIAL steps are hidden as a whole (diagonals, window and
    prefix edges, ragged ends), and with keys no query sees (columns of blocks without a step)."""
    import paper_2412_05496_amd as fa
    dev = torch.device(DEV)
    wl = wlm.CFG1.scaled(name="hidden", B=1, Hq=2, Hkv=Hkv, S=S + extra_keys, D=64, Bq=Bq, Bk=Bk, mask=mask, score=score,
                         window=40, prefix_len=70, softcap=20.0, rel_len=20, seed=4300 + S)
    inp = wlm.make_train_inputs(wl, with_dO=True)
    inp.Q, inp.dO = inp.Q[:, :, :S].contiguous(), inp.dO[:, :, :S].contiguous()
    score_mod, mask_mod = hp.oracle_mods(wl, inp)
    mask_id, score_id, params, _ = hp.library_mods(wl, inp, dev)
    print(f"[case] hidden blocks {mask} {score} S={S}+{extra_keys}", flush=True)
    bm = fa.alloc_blockmask(1, 1, S, S + extra_keys, Bq, Bk, device=dev)
    fa.flexattn_blockmask_build(mask_id, params, bm)
    Q, K, V = (t.to(dev) for t in (inp.Q, inp.K, inp.V))
    O, LSE = torch.full_like(Q, float("nan")), torch.full(Q.shape[:3], float("nan"), device=dev)
    fa.flexattn_forward(Q, K, V, score_id, mask_id, params, bm, inp.scale, O, LSE)
    torch.cuda.synchronize()
    ref = fo.flex_attention_backward(inp.Q, inp.K, inp.V, inp.dO, score_mod, mask_mod, inp.scale)
    for stored in (False, True):
        grads = hp.run_backward(wl, inp, dev, O, LSE, bm, (mask_id, score_id, params, Q, K, V), stored=stored)
        for name, got, r in zip(("dQ", "dK", "dV"), grads, ref):
            hp.check_grad(name, got, r)
        # 300 copies (batch stride 0): the forms for many workgroups
        n, hq = 300, Q.shape[1]
        Qn, Kn, Vn, On, dOn = (t.to(dev).expand(n, -1, -1, -1) for t in (Q, K, V, O, inp.dO))
        outs = [torch.full(t.shape, float("nan"), dtype=torch.bfloat16, device=dev) for t in (Qn, Kn, Vn)]
        args = (Qn, Kn, Vn, On, dOn, LSE.expand(n, hq, -1).contiguous(), score_id, mask_id, params, bm, inp.scale, *outs)
        if stored:
            fa.flexattn_backward_stored(*args, hp.nonempty_blocks(bm))
        else:
            fa.flexattn_backward(*args)
        torch.cuda.synchronize()
        for name, got, r in zip(("dQ", "dK", "dV"), outs, ref):
            hp.check_grad(name, got[:1], r)
            assert torch.equal(got, got[:1].expand_as(got)), name


@pytest.mark.parametrize("heads", [512, 520])
@pytest.mark.parametrize("mask,score", [("causal", "identity"), ("prefix_lm", "identity"), ("causal", "alibi_softcap"), ("none", "identity"),
                                        ("swa_causal_or_prefix", "rel_bias")])
def test_backward_d64_few_and_many_workgroups(mask, score, heads):
    """D = 64 gradients on both sides of the number of workgroups from which dQ leaves hidden blocks out (the one-head tests
    above take the forms of dK/dV and dQ for few workgroups).  The heads are the same (stride 0): one is compared with the
    oracle and the others with it."""
    import paper_2412_05496_amd as fa
    dev, S = torch.device(DEV), 100
    wl = wlm.CFG1.scaled(name="dq_sides", B=1, Hq=1, Hkv=1, S=S, D=64, Bq=128, Bk=64, mask=mask, score=score, prefix_len=70,
                         window=40, softcap=20.0, rel_len=20, seed=4350)
    inp = wlm.make_train_inputs(wl, with_dO=True)
    score_mod, mask_mod = hp.oracle_mods(wl, inp)
    mask_id, score_id, params, _ = hp.library_mods(wl, inp, dev)
    if params.alibi_bias is not None:
        params.alibi_bias = params.alibi_bias.repeat(heads)
    if params.rel_bias is not None:
        params.rel_bias = params.rel_bias.repeat(heads, 1)
    bm = fa.alloc_blockmask(1, 1, S, S, 128, 64, device=dev)
    fa.flexattn_blockmask_build(mask_id, params, bm)
    Q, K, V, dO = (t.to(dev).expand(1, heads, S, 64) for t in (inp.Q, inp.K, inp.V, inp.dO))
    O, LSE = torch.empty(Q.shape, dtype=torch.bfloat16, device=dev), torch.empty(Q.shape[:3], device=dev)
    fa.flexattn_forward(Q, K, V, score_id, mask_id, params, bm, inp.scale, O, LSE)
    dQ, dK, dV = (torch.full(Q.shape, float("nan"), dtype=torch.bfloat16, device=dev) for _ in range(3))
    fa.flexattn_backward(Q, K, V, O, dO, LSE, score_id, mask_id, params, bm, inp.scale, dQ, dK, dV)
    torch.cuda.synchronize()
    ref = fo.flex_attention_backward(inp.Q, inp.K, inp.V, inp.dO, score_mod, mask_mod, inp.scale)
    for name, got, r in zip(("dQ", "dK", "dV"), (dQ, dK, dV), ref):
        hp.check_grad(name, got[:, :1], r)
        assert torch.equal(got, got[:, :1].expand_as(got)), name


@pytest.mark.parametrize("w,h,k,layout,tile", [(200, 1, 1, "row_major", 0), (1, 130, 1, "row_major", 0),
                                               (15, 15, 15, "row_major", 0), (17, 9, 9, "row_major", 0),
                                               (24, 8, 7, "tiled", 4), (16, 16, 3, "morton", 0)])
def test_canvas_edges(w, h, k, layout, tile):
    import paper_2412_05496_amd as fa
    S, dev = w * h, torch.device(DEV)
    wl = wlm.CFG1.scaled(name="canvas", B=1, Hq=2, Hkv=2, S=S, D=64, Bq=128, Bk=64, seed=4200 + S)
    inp = wlm.make_train_inputs(wl, with_dO=True)
    mask_mod, score_mod = fo.neighborhood_mask(w, h, k, layout, tile), fo.Identity()
    params = fa.ModParams(na_width=w, na_height=h, na_kernel=k, na_tile=tile,
                          na_layout={"row_major": fa.NA_ROW_MAJOR, "tiled": fa.NA_TILED, "morton": fa.NA_MORTON}[layout])
    print(f"[case] canvas {w}x{h} K={k} {layout}", flush=True)
    bm = fa.alloc_blockmask(1, 1, S, S, wl.Bq, wl.Bk, device=dev)
    fa.flexattn_blockmask_build(fa.MASK_NEIGHBORHOOD, params, bm)
    torch.cuda.synchronize()
    hp.assert_blockmask_equal(bm, fo.create_block_mask(mask_mod, 1, 1, S, S, wl.Bq, wl.Bk))
    Q, K, V = (t.to(dev) for t in (inp.Q, inp.K, inp.V))
    O, LSE = torch.full_like(Q, float("nan")), torch.full(Q.shape[:3], float("nan"), device=dev)
    fa.flexattn_forward(Q, K, V, fa.SCORE_IDENTITY, fa.MASK_NEIGHBORHOOD, params, bm, inp.scale, O, LSE)
    torch.cuda.synchronize()
    hp.check_output(O, LSE, *fo.flex_attention(inp.Q, inp.K, inp.V, score_mod, mask_mod, inp.scale))
    ref = fo.flex_attention_backward(inp.Q, inp.K, inp.V, inp.dO, score_mod, mask_mod, inp.scale)
    ids = (fa.MASK_NEIGHBORHOOD, fa.SCORE_IDENTITY, params, Q, K, V)
    for stored in (False, True):
        for name, got, r in zip(("dQ", "dK", "dV"), hp.run_backward(wl, inp, dev, O, LSE, bm, ids, stored=stored), ref):
            hp.check_grad(name, got, r)


@pytest.mark.parametrize("w,h,k,layout,tile,Bq,Bk", [
    (33, 40, 5, "row_major", 0, 128, 64), (100, 9, 3, "row_major", 4, 64, 64), (40, 24, 7, "tiled", 8, 128, 64),
    (20, 44, 3, "tiled", 2, 128, 128), (24, 36, 5, "tiled", 4, 128, 64), (40, 24, 5, "tiled", 1, 128, 64),
    (48, 32, 5, "tiled", 16, 64, 128), (64, 32, 5, "tiled", 32, 128, 64), (32, 32, 9, "morton", 0, 128, 128)])
@pytest.mark.parametrize("D", [64, 128])
def test_canvas_blocks_left_out(w, h, k, layout, tile, Bq, Bk, D):
    """Canvases of several row blocks in every token order and tile size: the 32 x 32 blocks, tiles and steps
    that are left out because the windows cannot reach them."""
    import paper_2412_05496_amd as fa
    S, dev = w * h, torch.device(DEV)
    wl = wlm.CFG1.scaled(name="canvas_cut", B=1, Hq=2, Hkv=1, S=S, D=D, Bq=Bq, Bk=Bk, seed=4400 + S)
    inp = wlm.make_train_inputs(wl, with_dO=True)
    mask_mod, score_mod = fo.neighborhood_mask(w, h, k, layout, tile), fo.Identity()
    params = fa.ModParams(na_width=w, na_height=h, na_kernel=k, na_tile=tile,
                          na_layout={"row_major": fa.NA_ROW_MAJOR, "tiled": fa.NA_TILED, "morton": fa.NA_MORTON}[layout])
    print(f"[case] canvas blocks {w}x{h} K={k} {layout} T={tile} D={D}", flush=True)
    bm = fa.alloc_blockmask(1, 1, S, S, Bq, Bk, device=dev)
    fa.flexattn_blockmask_build(fa.MASK_NEIGHBORHOOD, params, bm)
    Q, K, V = (t.to(dev) for t in (inp.Q, inp.K, inp.V))
    O, LSE = torch.full_like(Q, float("nan")), torch.full(Q.shape[:3], float("nan"), device=dev)
    fa.flexattn_forward(Q, K, V, fa.SCORE_IDENTITY, fa.MASK_NEIGHBORHOOD, params, bm, inp.scale, O, LSE)
    torch.cuda.synchronize()
    hp.check_output(O, LSE, *fo.flex_attention(inp.Q, inp.K, inp.V, score_mod, mask_mod, inp.scale))
    ref = fo.flex_attention_backward(inp.Q, inp.K, inp.V, inp.dO, score_mod, mask_mod, inp.scale)
    ids = (fa.MASK_NEIGHBORHOOD, fa.SCORE_IDENTITY, params, Q, K, V)
    for stored in (False, True):
        for name, got, r in zip(("dQ", "dK", "dV"), hp.run_backward(wl, inp, dev, O, LSE, bm, ids, stored=stored), ref):
            hp.check_grad(name, got, r)


@pytest.mark.parametrize("q_len,kv_len,Bq,Bk", [(48, 4800, 8, 16), (2049, 70, 8, 16), (100, 257 * 5, 33, 5), (130, 200, 130, 200)])
def test_long_lines_and_odd_blocks(q_len, kv_len, Bq, Bk):
    """More than 256 blocks in a line (both orientations), block sizes above 64 that are no power of two,
    query offsets, and more than 256 lines to order."""
    import paper_2412_05496_amd as fa
    n = max(q_len, kv_len) + 40
    docs = scattered_ids(1, n, 3, seed=q_len)
    packed = wlm.document_ids([60, 37, 300] + [n - 397] if n > 397 else [n // 3, n - n // 3])[None, :].contiguous()
    off = torch.tensor([40], dtype=torch.int32)
    p = dict(q_offsets=off.to(DEV))
    cases = [(fa.MASK_DOCUMENT_CAUSAL, fa.ModParams(doc_ids=docs.to(DEV), **p), fo.and_mask(fo.document_mask(docs), fo.causal_mask)),
             (fa.MASK_DOCUMENT, fa.ModParams(doc_ids=packed.to(DEV), **p), fo.document_mask(packed)),
             (fa.MASK_SWA_CAUSAL_OR_PREFIX, fa.ModParams(window=30, prefix_len=19, **p),
              fo.or_mask(fo.and_mask(fo.causal_mask, fo.sliding_window_mask(30)), fo.prefix_mask(19)))]
    for mask_id, params, mod in cases:
        print(f"[case] mask {mask_id:#x} {q_len}x{kv_len} blocks {Bq}x{Bk}", flush=True)
        bm = fa.alloc_blockmask(1, 1, q_len, kv_len, Bq, Bk, device=DEV)
        for name in ("kv_indices", "full_kv_indices", "q_indices", "full_q_indices"):
            getattr(bm, name).fill_(-7)
        fa.flexattn_blockmask_build(mask_id, params, bm)
        torch.cuda.synchronize()
        hp.assert_blockmask_equal(bm, fo.create_block_mask(fo.with_q_offset(mod, off), 1, 1, q_len, kv_len, Bq, Bk))
