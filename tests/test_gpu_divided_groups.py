"""dK and dV of few KV heads, whose query heads are divided among workgroups: parts of one head and of several, of unlike size, in either kernel,
against the oracle; and the same launch with a workspace that has no room for the parts' sums."""
import pytest
import torch

from oracle import flex_oracle as fo
from tests import helpers as hp

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# B, Hq, Hkv, S, D, mask, Bq, Bk, per-head BlockMasks, parts
CASES = [
    (1, 4, 1, 709, 128, "causal", 128, 64, False, 4),
    (1, 3, 1, 1100, 128, "causal", 128, 64, False, 2),          # parts of one and two heads
    (2, 7, 1, 900, 64, "prefix", 128, 128, False, 4),           # of one, two, two and two
    (1, 8, 1, 2500, 64, "causal", 128, 64, False, 4),
    (2, 16, 2, 1500, 64, "documents", 128, 64, False, 4),       # 384 workgroups, not by slices of 32 keys
    (2, 16, 2, 1500, 128, "causal", 128, 64, False, 4),         # the same
    (1, 16, 4, 850, 128, "documents", 64, 64, False, 2),
    (1, 6, 2, 1500, 64, "window", 128, 64, True, 2),
    (1, 8, 1, 1024, 64, "neighborhood", 128, 64, False, 8),
    (1, 8, 1, 1024, 128, "none", 64, 128, True, 8),
]


def mods(fa, mask, S, B):
    params = fa.ModParams()
    if mask == "causal":
        return params, fa.MASK_CAUSAL, fo.causal_mask
    if mask == "none":
        return params, fa.MASK_NONE, fo.no_mask
    if mask == "window_or_prefix":
        params.window, params.prefix_len = 300, 50
        return params, fa.MASK_SWA_CAUSAL_OR_PREFIX, None
    if mask == "prefix":
        params.prefix_len = 70
        return params, fa.MASK_PREFIX_LM, fo.or_mask(fo.causal_mask, fo.prefix_mask(70))
    if mask == "window":
        params.window = 900
        return params, fa.MASK_SWA_CAUSAL, fo.and_mask(fo.causal_mask, fo.sliding_window_mask(900))
    if mask == "documents":
        ids = (torch.arange(S) >= S // 3).to(torch.int32).expand(B, S).contiguous()
        params.doc_ids = ids.to(DEV)
        return params, fa.MASK_DOCUMENT_CAUSAL, fo.and_mask(fo.document_mask(ids), fo.causal_mask)
    params.na_width, params.na_height, params.na_kernel, params.na_layout, params.na_tile = 32, 32, 21, fa.NA_TILED, 8
    return params, fa.MASK_NEIGHBORHOOD, fo.neighborhood_mask(32, 32, 21, "tiled", 8)


@pytest.mark.parametrize("B,Hq,Hkv,S,D,mask,Bq,Bk,per_head,parts", CASES)
def test_divided_groups(B, Hq, Hkv, S, D, mask, Bq, Bk, per_head, parts):
    import paper_2412_05496_amd as fa
    print("[case]", B, Hq, Hkv, S, D, mask, Bq, Bk, flush=True)
    gen = torch.Generator().manual_seed(S + Hq)
    Q, dO = (torch.randn(B, Hq, S, D, generator=gen).to(torch.bfloat16) for _ in range(2))
    K, V = (torch.randn(B, Hkv, S, D, generator=gen).to(torch.bfloat16) for _ in range(2))
    params, mask_id, oracle_mask = mods(fa, mask, S, B)
    scale = D ** -0.5
    bm = fa.alloc_blockmask(B if per_head or mask == "documents" else 1, Hq if per_head else 1, S, S, Bq, Bk, device=DEV)
    fa.flexattn_blockmask_build(mask_id, params, bm)
    q, k, v, do = (t.to(DEV) for t in (Q, K, V, dO))
    O, LSE = torch.empty_like(q), torch.empty(B, Hq, S, device=DEV)
    head = (fa.SCORE_IDENTITY, mask_id, params, bm, scale)
    fa.flexattn_forward(q, k, v, *head, O, LSE)
    scalars = 2 * B * Hq * S * 4
    at_most = (fa.flexattn_backward_workspace_bytes(q, k) - scalars) // (2 * B * Hkv * S * D * 4)
    assert at_most >= parts                                     # (whatever the mask)
    ref = fo.flex_attention_backward(Q, K, V, dO, fo.Identity(), oracle_mask, scale)
    got = []
    for room in (fa.flexattn_backward_workspace_bytes(q, k), scalars):
        ws = torch.full((room + 4096,), 0xFF, dtype=torch.uint8, device=DEV)
        # rows of every other head's storage, [B, S, H, D]
        dQ, dK, dV = (torch.full((B, S, t.shape[1], D), float("nan"), dtype=torch.bfloat16, device=DEV).transpose(1, 2) for t in (q, k, k))
        fa.flexattn_backward(q, k, v, O, do, LSE, *head, dQ, dK, dV, ws[:room])
        torch.cuda.synchronize()
        for name, g, r in zip(("dQ", "dK", "dV"), (dQ, dK, dV), ref):
            hp.check_grad(name, g, r)
        assert bool((ws[room:] == 0xFF).all())
        written = int((ws[:room].view(torch.int32) != -1).sum()) * 4 - scalars
        # the parts of this mask; the sums are hardly ever NaN patterns
        assert room == scalars or abs(written / (2 * B * Hkv * S * D * 4) - parts) < 0.01, written / (2 * B * Hkv * S * D * 4)
        got.append((dK, dV))
    # the same products, added up in another order in fp32: one bf16 rounding of each result
    for a, b in zip(*got):
        assert (a.float() - b.float()).abs().max() <= 2 ** -7 * b.float().abs().max()
    # with dS in memory, bit for bit, by stages and with no more room than whole groups need
    n = hp.nonempty_blocks(bm)
    need = fa.flexattn_backward_stored_workspace_bytes(q, k, bm, n)
    for room, want in ((need, got[0]), (need - hp.room_for_parts(q, k), got[1])):
        ws = torch.full((room,), 0xFF, dtype=torch.uint8, device=DEV)
        dQ, dK, dV = (torch.full_like(t, float("nan")) for t in (q, k, k))
        for stages in (1, 2, 4):
            fa.flexattn_backward_stored(q, k, v, O, do, LSE, *head, dQ, dK, dV, n, ws, stages)
        torch.cuda.synchronize()
        hp.check_grad("dQ*", dQ, ref[0])
        assert torch.equal(dK, want[0]) and torch.equal(dV, want[1])
    with pytest.raises(fa.FlexAttnError):
        fa.flexattn_backward(q, k, v, O, do, LSE, *head, dQ, dK, dV, ws[:scalars - 4])


def test_stages_with_workspaces_of_different_sizes():
    """Where the block numbers and dS lie does not depend on whether the workspace has room for the parts' sums: every stage may be
    told of it or not.  (dQ first: the others' blocks at other places would be read, within the workspace.)"""
    import paper_2412_05496_amd as fa
    B, Hq, Hkv, S, D = 1, 4, 1, 709, 128
    gen = torch.Generator().manual_seed(5)
    Q, dO = (torch.randn(B, Hq, S, D, generator=gen).to(torch.bfloat16) for _ in range(2))
    K, V = (torch.randn(B, Hkv, S, D, generator=gen).to(torch.bfloat16) for _ in range(2))
    bm = fa.alloc_blockmask(1, 1, S, S, 128, 64, device=DEV)
    params = fa.ModParams()
    fa.flexattn_blockmask_build(fa.MASK_CAUSAL, params, bm)
    q, k, v, do = (t.to(DEV) for t in (Q, K, V, dO))
    O, LSE = torch.empty_like(q), torch.empty(B, Hq, S, device=DEV)
    head = (fa.SCORE_IDENTITY, fa.MASK_CAUSAL, params, bm, D ** -0.5)
    fa.flexattn_forward(q, k, v, *head, O, LSE)
    ref = fo.flex_attention_backward(Q, K, V, dO, fo.Identity(), fo.causal_mask, D ** -0.5)
    n = hp.nonempty_blocks(bm)
    need, less = fa.flexattn_backward_stored_workspace_bytes(q, k, bm, n), hp.room_for_parts(q, k)
    assert less > 0
    first = None
    for lacking in (4, 0, 7, 3, 2, 5, 1, 6):                # the stages (a bit each) whose workspace lacks the room
        print("[case] lacking", lacking, flush=True)
        ws = torch.full((need,), 0xFF, dtype=torch.uint8, device=DEV)
        dQ, dK, dV = (torch.full_like(t, float("nan")) for t in (q, k, k))
        for stage in (1, 2, 4):
            fa.flexattn_backward_stored(q, k, v, O, do, LSE, *head, dQ, dK, dV, n, ws[:need - less] if lacking & stage else ws, stage)
        torch.cuda.synchronize()
        for name, g, r in zip(("dQ", "dK", "dV"), (dQ, dK, dV), ref):
            hp.check_grad(name, g, r)
        first = dQ if first is None else first
        assert torch.equal(dQ, first)


# B, Hq, Hkv, S, D, length of the documents of plane 0 and of the others, the orders of the BlockMask are there, parts of the sums
DOCUMENTS = [
    (8, 2, 1, 2048, 128, 40, 40, True, 0),          # asked: the longest column is short, whole groups
    (8, 2, 1, 2048, 128, 2048, 40, True, 2),        # asked: long
    (8, 2, 1, 2048, 128, 40, 2048, True, 0),        # (the first plane's columns are asked for all)
    (8, 2, 1, 2048, 128, 2048, 2048, False, 0),     # nothing says which column is the longest: whole
    (2, 12, 3, 4000, 128, 30, 60, True, 0),         # asked, of four heads
    (2, 12, 3, 4000, 128, 700, 300, True, 2),
    (3, 4, 2, 4096, 64, 90, 90, True, 0),           # asked, 768 workgroups
    (3, 4, 2, 4096, 64, 900, 90, True, 2),
    (1, 8, 1, 900, 64, 50, 50, True, 8),            # so few keys that short ones do not lose
]


@pytest.mark.parametrize("B,Hq,Hkv,S,D,first,others,orders,parts", DOCUMENTS)
def test_documents(B, Hq, Hkv, S, D, first, others, orders, parts):
    """Launches that divide the groups of long documents and leave those of short ones whole."""
    import paper_2412_05496_amd as fa
    print("[case]", B, Hq, Hkv, S, D, first, others, orders, flush=True)
    gen = torch.Generator().manual_seed(S + Hq)
    Q, dO = (torch.randn(B, Hq, S, D, generator=gen).to(torch.bfloat16) for _ in range(2))
    K, V = (torch.randn(B, Hkv, S, D, generator=gen).to(torch.bfloat16) for _ in range(2))
    ids = torch.stack([torch.arange(S, dtype=torch.int32) // (others if b else first) for b in range(B)])
    params = fa.ModParams()
    params.doc_ids = ids.to(DEV)
    bm = fa.alloc_blockmask(B, 1, S, S, 128, 64, device=DEV)
    fa.flexattn_blockmask_build(fa.MASK_DOCUMENT_CAUSAL, params, bm)
    if not orders:
        bm.kv_order = bm.q_order = None
    q, k, v, do = (t.to(DEV) for t in (Q, K, V, dO))
    O, LSE = torch.empty_like(q), torch.empty(B, Hq, S, device=DEV)
    head = (fa.SCORE_IDENTITY, fa.MASK_DOCUMENT_CAUSAL, params, bm, D ** -0.5)
    fa.flexattn_forward(q, k, v, *head, O, LSE)
    room, scalars = fa.flexattn_backward_workspace_bytes(q, k), 2 * B * Hq * S * 4
    one = 2 * B * Hkv * S * D * 4
    assert room - scalars >= max(parts, 2) * one
    n, got = hp.nonempty_blocks(bm), []
    for stored in (False, True):
        ws = hp.dirty_stored_workspace(q, k, bm, n) if stored else torch.full((room,), 0xFF, dtype=torch.uint8, device=DEV)
        dQ, dK, dV = (torch.full_like(t, float("nan")) for t in (q, k, k))
        for stage in (1, 2, 4):
            if stored:
                fa.flexattn_backward_stored(q, k, v, O, do, LSE, *head, dQ, dK, dV, n, ws, stage)
            else:
                fa.flexattn_backward_stages(q, k, v, O, do, LSE, *head, dQ, dK, dV, ws, stage)
        torch.cuda.synchronize()
        sums = ws[ws.numel() - hp.room_for_parts(q, k):]
        written = int((sums.view(torch.int32) != -1).sum()) * 4 / one
        assert abs(written - parts) < 0.01, written
        got.append((dQ, dK, dV))
    assert torch.equal(got[0][1], got[1][1]) and torch.equal(got[0][2], got[1][2])
    for b in sorted({0, B - 1}):            # (an entry at a time, document by document: the oracle's scores are S x S)
        for lo in range(0, S, others if b else first):
            hi = min(lo + (others if b else first), S)
            if lo and hi < S and lo % 3:    # (a third of them, the first and the last)
                continue
            cut = [t[b:b + 1, :, lo:hi].float() for t in (Q, K, V, dO)]
            ref = fo.flex_attention_backward(*cut, fo.Identity(), fo.causal_mask, D ** -0.5)
            for grads in got:
                for name, g, r in zip(("dQ", "dK", "dV"), grads, ref):
                    hp.check_grad(name, g[b:b + 1, :, lo:hi], r)
    for t in (x for grads in got for x in grads):
        assert bool(torch.isfinite(t).all())


# B, Hq, Hkv, S, D, mask: groups that stay whole, though they have heads and steps enough
WHOLE = [
    (1, 6, 2, 4000, 64, "none"),            # unlike parts
    (4, 9, 3, 1000, 128, "causal"),
    (1, 4, 2, 4000, 64, "none"),            # split among the waves, which two parts would not be
    (1, 64, 8, 1000, 64, "none"),
    (1, 12, 3, 1500, 64, "causal"),         # one head each
    (1, 40, 8, 2048, 64, "window_or_prefix"),       # unlike parts, split in either case
]


@pytest.mark.parametrize("B,Hq,Hkv,S,D,mask", WHOLE)
def test_groups_that_stay_whole(B, Hq, Hkv, S, D, mask):
    import paper_2412_05496_amd as fa
    print("[case]", B, Hq, Hkv, S, D, mask, flush=True)
    q, k, v, do = (torch.randn(B, h, S, D, device=DEV).to(torch.bfloat16) for h in (Hq, Hkv, Hkv, Hq))
    params, mask_id, _ = mods(fa, mask, S, B)
    bm = fa.alloc_blockmask(1, 1, S, S, 128, 64, device=DEV)
    fa.flexattn_blockmask_build(mask_id, params, bm)
    O, LSE = torch.empty_like(q), torch.empty(B, Hq, S, device=DEV)
    head = (fa.SCORE_REL_BIAS if mask == "window_or_prefix" else fa.SCORE_IDENTITY, mask_id, params, bm, D ** -0.5)
    params.rel_bias = torch.zeros(Hq, 16, device=DEV)
    fa.flexattn_forward(q, k, v, *head, O, LSE)
    scalars, got = 2 * B * Hq * S * 4, []
    for room in (fa.flexattn_backward_workspace_bytes(q, k), scalars):
        ws = torch.full((room,), 0xFF, dtype=torch.uint8, device=DEV)
        dQ, dK, dV = (torch.full_like(t, float("nan")) for t in (q, k, k))
        fa.flexattn_backward(q, k, v, O, do, LSE, *head, dQ, dK, dV, ws)
        assert bool((ws[scalars:] == 0xFF).all())
        got.append((dK, dV))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("D,score", [(64, "softcap"), (128, "softcap"), (64, "alibi"), (128, "alibi"), (64, "alibi_softcap"), (128, "rel_bias"), (64, "rel_bias")])
def test_divided_groups_with_a_score_mod(D, score):
    """The factor of a soft-cap's derivative belongs to dK's sums and not to dV's."""
    import paper_2412_05496_amd as fa
    print("[case]", D, score, flush=True)
    B, Hq, Hkv, S = 1, 8, 1, 1100
    gen = torch.Generator().manual_seed(D)
    Q, dO = (torch.randn(B, Hq, S, D, generator=gen).to(torch.bfloat16) for _ in range(2))
    K, V = (torch.randn(B, Hkv, S, D, generator=gen).to(torch.bfloat16) for _ in range(2))
    bias, table = -2.0 ** -torch.arange(1.0, Hq + 1), 0.3 * torch.randn(Hq, 90, generator=gen)
    params, mask_id, mask = mods(fa, "causal", S, B)
    params.softcap, params.alibi_bias, params.rel_bias = 20.0, bias.to(DEV), table.to(DEV)
    alibi, cap = fo.Alibi(bias.double()), fo.Softcap(20.0)
    if score == "rel_bias":         # (compiled with a window or a prefix)
        params.window, params.prefix_len, mask_id = 900, 40, fa.MASK_SWA_CAUSAL_OR_PREFIX
        mask = fo.or_mask(fo.and_mask(fo.causal_mask, fo.sliding_window_mask(900)), fo.prefix_mask(40))
    score_id, score_mod = {"softcap": (fa.SCORE_SOFTCAP, cap), "alibi": (fa.SCORE_ALIBI, alibi), "rel_bias": (fa.SCORE_REL_BIAS, fo.RelBias(table.double())),
                           "alibi_softcap": (fa.SCORE_ALIBI | fa.SCORE_SOFTCAP, fo.Compose(alibi, cap))}[score]
    bm = fa.alloc_blockmask(1, 1, S, S, 128, 64, device=DEV)
    fa.flexattn_blockmask_build(mask_id, params, bm)
    q, k, v, do = (t.to(DEV) for t in (Q, K, V, dO))
    O, LSE = torch.empty_like(q), torch.empty(B, Hq, S, device=DEV)
    head = (score_id, mask_id, params, bm, D ** -0.5)
    fa.flexattn_forward(q, k, v, *head, O, LSE)
    ws = torch.full((fa.flexattn_backward_workspace_bytes(q, k),), 0xFF, dtype=torch.uint8, device=DEV)
    grads = [torch.full_like(t, float("nan")) for t in (q, k, k)]
    fa.flexattn_backward(q, k, v, O, do, LSE, *head, *grads, ws)
    assert bool((ws[ws.numel() - hp.room_for_parts(q, k):] != 0xFF).any())          # (divided)
    for name, g, r in zip(("dQ", "dK", "dV"), grads, fo.flex_attention_backward(Q, K, V, dO, score_mod, mask, D ** -0.5)):
        hp.check_grad(name, g, r)


@pytest.mark.parametrize("B,Hq,Hkv,S,D", [(8, 2, 1, 2048, 128), (3, 4, 2, 4096, 64)])
def test_documents_that_change_between_replays(B, Hq, Hkv, S, D):
    """The question is asked on the device, of the lists as they are when a captured step runs: short documents and long ones in turn."""
    import paper_2412_05496_amd as fa
    print("[case] replays", B, Hq, Hkv, S, D, flush=True)
    gen = torch.Generator().manual_seed(S)
    q, do = (torch.randn(B, Hq, S, D, generator=gen).to(torch.bfloat16).to(DEV) for _ in range(2))
    k, v = (torch.randn(B, Hkv, S, D, generator=gen).to(torch.bfloat16).to(DEV) for _ in range(2))
    params = fa.ModParams()
    params.doc_ids = torch.zeros(B, S, dtype=torch.int32, device=DEV)
    bm = fa.alloc_blockmask(B, 1, S, S, 128, 64, device=DEV)
    bm_ws = torch.empty(max(fa.flexattn_blockmask_workspace_bytes(B, 1, S, S, 128, 64), 1), dtype=torch.uint8, device=DEV)
    O, LSE = torch.empty_like(q), torch.empty(B, Hq, S, device=DEV)
    grads = [torch.empty_like(t) for t in (q, k, k)]
    ws = torch.empty(fa.flexattn_backward_workspace_bytes(q, k), dtype=torch.uint8, device=DEV)
    head = (fa.SCORE_IDENTITY, fa.MASK_DOCUMENT_CAUSAL, params, bm, D ** -0.5)

    def step():
        fa.flexattn_blockmask_build(fa.MASK_DOCUMENT_CAUSAL, params, bm, bm_ws)
        fa.flexattn_forward(q, k, v, *head, O, LSE)
        fa.flexattn_backward(q, k, v, O, do, LSE, *head, *grads, ws)

    def load(length):
        params.doc_ids.copy_((torch.arange(S, dtype=torch.int32) // length).expand(B, S))

    def parts_written():
        return bool((ws[ws.numel() - hp.room_for_parts(q, k):] != 0xFF).any())

    lengths, eager = (50, 1500, 90, 700), []
    for n in lengths:
        load(n)
        ws.fill_(0xFF)
        step()
        torch.cuda.synchronize()
        assert parts_written() == (n > 100)
        eager.append([t.clone() for t in grads])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for _ in range(2):
        for n, want in zip(lengths, eager):
            load(n)
            ws.fill_(0xFF)
            for t in grads:
                t.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert parts_written() == (n > 100)
            for got, ref in zip(grads, want):
                assert torch.equal(got, ref)
            (torch.randn(256, 256, device=DEV) @ torch.randn(256, 256, device=DEV)).sum().item()       # eager work between the replays
