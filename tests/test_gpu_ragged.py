"""GPU parity for sequence lengths that are no multiple of the block size: the last row / column of
BlockMask blocks is cut by the edge of the score matrix (BlockMask bit for bit, forward, backward)."""
import pytest
import torch

import flex_workloads as wlm
from oracle import flex_oracle as fo
from tests import helpers as hp

pytestmark = pytest.mark.gpu

CASES = [
    # name, base workload, overrides, q_len (None = S)
    ("causal_softcap_d128_s1000", wlm.CFG2, dict(B=1, Hq=2, Hkv=2, S=1000), None),
    ("none_d64_300x777_bk128", wlm.CFG1, dict(B=1, Hq=2, Hkv=1, S=777, D=64, Bq=64, Bk=128, mask="none", backward=True), 300),
    ("causal_d64_q1_kv65", wlm.CFG1, dict(B=2, Hq=2, Hkv=2, S=65, backward=True), 1),
    ("doc_alibi_d64_s1000", wlm.CFG3, dict(B=2, Hq=4, Hkv=4, S=1000, doc_len_min=50, doc_len_max=400), None),
    ("swa_prefix_relbias_gqa_d128_s999", wlm.CFG4, dict(B=1, Hq=4, Hkv=2, S=999, window=200, prefix_len=100, rel_len=64), None),
    ("causal_d128_s130_bq128", wlm.CFG2, dict(B=1, Hq=1, Hkv=1, S=130, score="identity"), None),
]


# D = 128 forward, few workgroups: 64-key tiles (rows of 1, 2, 3 tiles, short and long)
CASES += [(f"{mask}_{score}_d128_s{S}", wlm.CFG2, dict(B=1, Hq=1, Hkv=1, S=S, mask=mask, score=score), q_len)
          for mask, score, S, q_len in [("none", "identity", 33, None), ("none", "identity", 100, 70), ("none", "identity", 190, 20),
                                        ("causal", "identity", 1536, None), ("causal", "identity", 1537, None),
                                        ("none", "identity", 1601, 200), ("causal", "softcap", 1540, 130)]]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_ragged_lengths(case):
    import paper_2412_05496_amd as fa
    name, base, over, q_len = case
    dev = torch.device("cuda:0")
    wl = base.scaled(name="ragged_" + name, seed=3500 + len(name), **over)
    inp = wlm.make_train_inputs(wl, with_dO=True)
    Lq = wl.S if q_len is None else q_len
    Q, dO = inp.Q[:, :, :Lq].contiguous(), inp.dO[:, :, :Lq].contiguous()
    score_mod, mask_mod = hp.oracle_mods(wl, inp)
    O_ref, LSE_ref = fo.flex_attention(Q, inp.K, inp.V, score_mod, mask_mod, inp.scale)
    dQ_ref, dK_ref, dV_ref = fo.flex_attention_backward(Q, inp.K, inp.V, dO, score_mod, mask_mod, inp.scale)

    mask_id, score_id, params, Bm = hp.library_mods(wl, inp, dev)
    bm = fa.alloc_blockmask(Bm, 1, Lq, wl.S, wl.Bq, wl.Bk, device=dev)
    fa.flexattn_blockmask_build(mask_id, params, bm)
    torch.cuda.synchronize()
    hp.assert_blockmask_equal(bm, fo.create_block_mask(mask_mod, Bm, 1, Lq, wl.S, wl.Bq, wl.Bk))

    # guard rows / keys right behind the tensors: the kernels must not write past the real lengths
    def padded(t, rows):
        buf = torch.full((t.shape[0], t.shape[1], rows + 64, t.shape[3]), 7.0, dtype=t.dtype, device=dev)
        return buf, buf[:, :, :rows]
    Qd, Kd, Vd, dOd = Q.to(dev), inp.K.to(dev), inp.V.to(dev), dO.to(dev)
    O_buf, O = padded(Qd, Lq)
    dQ_buf, dQ = padded(Qd, Lq)
    dK_buf, dK = padded(Kd, wl.S)
    dV_buf, dV = padded(Vd, wl.S)
    LSE = torch.full(Qd.shape[:3], float("nan"), dtype=torch.float32, device=dev)
    fa.flexattn_forward(Qd, Kd, Vd, score_id, mask_id, params, bm, inp.scale, O, LSE)
    fa.flexattn_backward(Qd, Kd, Vd, O, dOd, LSE, score_id, mask_id, params, bm, inp.scale, dQ, dK, dV)
    torch.cuda.synchronize()
    hp.check_output(O, LSE, O_ref, LSE_ref)
    hp.check_grad("dQ", dQ, dQ_ref)
    hp.check_grad("dK", dK, dK_ref)
    hp.check_grad("dV", dV, dV_ref)
    for buf, rows in ((O_buf, Lq), (dQ_buf, Lq), (dK_buf, wl.S), (dV_buf, wl.S)):
        assert (buf[:, :, rows:] == 7.0).all()


@pytest.mark.parametrize("mask,score,S,q_len", [
    ("none", "identity", 33, None), ("none", "identity", 100, 70), ("none", "identity", 190, 20), ("causal", "identity", 257, None),
    ("causal", "softcap", 130, None), ("swa_causal", "identity", 300, None), ("swa_causal", "softcap", 200, None),
    ("causal", "alibi", 190, None), ("swa_causal_or_prefix", "rel_bias", 260, None), ("doc_causal", "alibi", 200, None)])
def test_forward_d128_many_workgroups(mask, score, S, q_len):
    """D = 128 forward with enough workgroups for 32-key units: rows of 1, 2, 3 ... units, every mask kind.  All
    sequences are the same (batch stride 0), so one is compared with the oracle and the others with it."""
    import paper_2412_05496_amd as fa
    dev, Lq = torch.device("cuda:0"), q_len or S
    wl = wlm.CFG2.scaled(name="units", B=1, Hq=2, Hkv=1, S=S, mask=mask, score=score, window=50, prefix_len=40, rel_len=30,
                         doc_len_min=30, doc_len_max=90, seed=3900 + S)
    inp = wlm.make_train_inputs(wl)
    score_mod, mask_mod = hp.oracle_mods(wl, inp)
    O_ref, LSE_ref = fo.flex_attention(inp.Q[:, :, :Lq], inp.K, inp.V, score_mod, mask_mod, inp.scale)
    mask_id, score_id, params, _ = hp.library_mods(wl, inp, dev)
    if params.doc_ids is not None:
        params.doc_ids = params.doc_ids[0].contiguous()
    bm = fa.alloc_blockmask(1, 1, Lq, S, wl.Bq, wl.Bk, device=dev)
    fa.flexattn_blockmask_build(mask_id, params, bm)
    B = 2304 // (2 * ((Lq + wl.Bq - 1) // wl.Bq)) + 1
    Q, K, V = (t.to(dev).expand(B, -1, -1, -1) for t in (inp.Q[:, :, :Lq].contiguous(), inp.K, inp.V))
    O = torch.full((B, 2, Lq, wl.D), float("nan"), dtype=torch.bfloat16, device=dev)
    LSE = torch.full((B, 2, Lq), float("nan"), device=dev)
    fa.flexattn_forward(Q, K, V, score_id, mask_id, params, bm, inp.scale, O, LSE)
    torch.cuda.synchronize()
    hp.check_output(O[:1], LSE[:1], O_ref, LSE_ref)
    assert torch.equal(O, O[:1].expand_as(O)) and torch.equal(LSE, LSE[:1].expand_as(LSE))


@pytest.mark.parametrize("w,h,k,layout,tile", [(40, 24, 7, "tiled", 8), (33, 20, 5, "row_major", 0), (32, 32, 9, "morton", 0)])
def test_forward_d128_canvas_many_workgroups(w, h, k, layout, tile):
    import paper_2412_05496_amd as fa
    dev, S = torch.device("cuda:0"), w * h
    wl = wlm.CFG2.scaled(name="units_canvas", B=1, Hq=2, Hkv=2, S=S, mask="none", score="identity", seed=3950 + S)
    inp = wlm.make_train_inputs(wl)
    params = fa.ModParams(na_width=w, na_height=h, na_kernel=k, na_tile=tile,
                          na_layout={"row_major": fa.NA_ROW_MAJOR, "tiled": fa.NA_TILED, "morton": fa.NA_MORTON}[layout])
    bm = fa.alloc_blockmask(1, 1, S, S, wl.Bq, wl.Bk, device=dev)
    fa.flexattn_blockmask_build(fa.MASK_NEIGHBORHOOD, params, bm)
    B = 2304 // (2 * ((S + wl.Bq - 1) // wl.Bq)) + 1
    Q, K, V = (t.to(dev).expand(B, -1, -1, -1) for t in (inp.Q, inp.K, inp.V))
    O = torch.full((B, 2, S, wl.D), float("nan"), dtype=torch.bfloat16, device=dev)
    LSE = torch.full((B, 2, S), float("nan"), device=dev)
    fa.flexattn_forward(Q, K, V, fa.SCORE_IDENTITY, fa.MASK_NEIGHBORHOOD, params, bm, inp.scale, O, LSE)
    torch.cuda.synchronize()
    hp.check_output(O[:1], LSE[:1], *fo.flex_attention(inp.Q, inp.K, inp.V, fo.Identity(), fo.neighborhood_mask(w, h, k, layout, tile), inp.scale))
    assert torch.equal(O, O[:1].expand_as(O)) and torch.equal(LSE, LSE[:1].expand_as(LSE))


@pytest.mark.parametrize("groups", [512, 544, 768, 800, 1248, 1280])
@pytest.mark.parametrize("mask,score,window", [("swa_causal", "identity", 100), ("swa_causal", "softcap", 200),
                                               ("swa_causal_or_prefix", "rel_bias", 90)])
def test_forward_d128_window_rounds(mask, score, window, groups):
    """Both sides of the numbers of workgroups, and windows up to and above half of the keys, between which the window
    masks change form at D = 128.  All sequences are the same (batch stride 0)."""
    import paper_2412_05496_amd as fa
    dev, S = torch.device("cuda:0"), 256
    wl = wlm.CFG2.scaled(name="rounds", B=1, Hq=2, Hkv=1, S=S, mask=mask, score=score, window=window, prefix_len=38, rel_len=30, seed=3970)
    inp = wlm.make_train_inputs(wl)
    score_mod, mask_mod = hp.oracle_mods(wl, inp)
    mask_id, score_id, params, _ = hp.library_mods(wl, inp, dev)
    bm = fa.alloc_blockmask(1, 1, S, S, wl.Bq, wl.Bk, device=dev)
    fa.flexattn_blockmask_build(mask_id, params, bm)
    B = groups // 4                 # (two heads of two row blocks each)
    Q, K, V = (t.to(dev).expand(B, -1, -1, -1) for t in (inp.Q, inp.K, inp.V))
    O = torch.full((B, 2, S, wl.D), float("nan"), dtype=torch.bfloat16, device=dev)
    LSE = torch.full((B, 2, S), float("nan"), device=dev)
    fa.flexattn_forward(Q, K, V, score_id, mask_id, params, bm, inp.scale, O, LSE)
    torch.cuda.synchronize()
    hp.check_output(O[:1], LSE[:1], *fo.flex_attention(inp.Q, inp.K, inp.V, score_mod, mask_mod, inp.scale))
    assert torch.equal(O, O[:1].expand_as(O)) and torch.equal(LSE, LSE[:1].expand_as(LSE))


def many(t, n):
    return t.repeat(n, *[1] * (t.dim() - 1))


@pytest.mark.parametrize("mask,score", [("swa_causal", "identity"), ("causal", "alibi"), ("doc_causal", "identity"), ("swa_causal", "softcap")])
@pytest.mark.parametrize("Bk", [64, 128])
def test_forward_d128_many_workgroups_planes_and_offsets(mask, score, Bk):
    """32-key units with a BlockMask plane per sequence, query offsets and two or four units to a block."""
    import paper_2412_05496_amd as fa
    dev, S, Lq, n = torch.device("cuda:0"), 500, 200, 97
    wl = wlm.CFG2.scaled(name="units_planes", B=3, Hq=4, Hkv=2, S=S, Bk=Bk, mask=mask, score=score, window=70, doc_len_min=30,
                         doc_len_max=200, seed=3980)
    inp = wlm.make_train_inputs(wl)
    off = torch.tensor([300, 111, 0], dtype=torch.int32)
    score_mod, mask_mod = hp.oracle_mods(wl, inp)
    score_mod, mask_mod = fo.QOffset(score_mod, off), fo.with_q_offset(mask_mod, off)
    mask_id, score_id, params, _ = hp.library_mods(wl, inp, dev)
    params.q_offsets = many(off, n).to(dev)
    if params.doc_ids is not None:
        params.doc_ids = many(params.doc_ids, n).contiguous()
    bm = fa.alloc_blockmask(3 * n, 1, Lq, S, wl.Bq, Bk, device=dev)
    fa.flexattn_blockmask_build(mask_id, params, bm)
    Q, K, V = (many(t, n).to(dev) for t in (inp.Q[:, :, :Lq].contiguous(), inp.K, inp.V))
    O = torch.full_like(Q, float("nan"))
    LSE = torch.full(Q.shape[:3], float("nan"), device=dev)
    fa.flexattn_forward(Q, K, V, score_id, mask_id, params, bm, inp.scale, O, LSE)
    torch.cuda.synchronize()
    hp.check_output(O[:3], LSE[:3], *fo.flex_attention(inp.Q[:, :, :Lq], inp.K, inp.V, score_mod, mask_mod, inp.scale))
    assert torch.equal(O, many(O[:3], n)) and torch.equal(LSE, many(LSE[:3], n))


@pytest.mark.parametrize("mask,score,S,q_len,B", [
    ("causal", "identity", 4095, 160, 1), ("causal", "identity", 4096, 160, 1), ("none", "identity", 4100, 90, 1),
    ("prefix_lm", "identity", 4200, 130, 1), ("causal", "alibi", 4097, 33, 1), ("causal", "alibi", 4097, 130, 700),
    ("causal", "softcap", 2047, 130, 1), ("causal", "softcap", 2050, 130, 1), ("causal", "alibi_softcap", 2048, 200, 1)])
def test_forward_d64_long_rows(mask, score, S, q_len, B):
    """D = 64 without windows: lengths on both sides of those at which the forward keeps its tile pipeline (soft-caps: too large
    to serve as the maximum), in launches so small that they are split, and one large one, plain by its number of workgroups
    (tests/test_gpu_forward_pipelined.py has the pipeline).  The queries are the last of the sequence."""
    import paper_2412_05496_amd as fa
    dev = torch.device("cuda:0")
    wl = wlm.CFG1.scaled(name="long_rows", B=1, Hq=2, Hkv=1, S=S, D=64, Bq=128, Bk=64, mask=mask, score=score, prefix_len=100, softcap=60.0,
                         seed=3990 + S)
    inp = wlm.make_train_inputs(wl)
    score_mod, mask_mod = hp.oracle_mods(wl, inp)
    off = torch.tensor([S - q_len], dtype=torch.int32)
    score_mod, mask_mod = fo.QOffset(score_mod, off), fo.with_q_offset(mask_mod, off)
    mask_id, score_id, params, _ = hp.library_mods(wl, inp, dev)
    params.q_offsets = off.repeat(B).to(dev)
    bm = fa.alloc_blockmask(1, 1, q_len, S, 128, 64, device=dev)
    fa.flexattn_blockmask_build(mask_id, params, bm)
    Q, K, V = (t.to(dev).expand(B, -1, -1, -1) for t in (inp.Q[:, :, -q_len:].contiguous(), inp.K, inp.V))
    O = torch.full(Q.shape, float("nan"), dtype=torch.bfloat16, device=dev)
    LSE = torch.full(Q.shape[:3], float("nan"), device=dev)
    fa.flexattn_forward(Q, K, V, score_id, mask_id, params, bm, inp.scale, O, LSE)
    torch.cuda.synchronize()
    hp.check_output(O[:1], LSE[:1], *fo.flex_attention(inp.Q[:, :, -q_len:], inp.K, inp.V, score_mod, mask_mod, inp.scale))
    assert torch.equal(O, O[:1].expand_as(O)) and torch.equal(LSE, LSE[:1].expand_as(LSE))
