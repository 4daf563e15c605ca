"""dQ from dS in memory where one workgroup takes two rows of blocks, or the same row of two heads, and their K tiles once: keys
that only one of the two rows lists, and lists longer than the 512 columns (or tiles) that the kernel takes at a time."""
import pytest
import torch

from tests import helpers as hp

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
D = 128


def tensors(B, Hq, Hkv, q_len, kv_len, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    return [torch.randn(B, h, n, D, generator=gen, device=DEV).to(torch.bfloat16) for h, n in ((Hq, q_len), (Hkv, kv_len), (Hkv, kv_len), (Hq, q_len))]


def backward(score_id, mask_id, params, bm, Q, K, V, dO, stored):
    import paper_2412_05496_amd as fa
    head = (score_id, mask_id, params, bm, D ** -0.5)
    O, LSE = torch.empty_like(Q), torch.empty(Q.shape[:3], dtype=torch.float32, device=DEV)
    fa.flexattn_forward(Q, K, V, *head, O, LSE)
    grads = [torch.full_like(t, float("nan")) for t in (Q, K, V)]
    if not stored:
        fa.flexattn_backward(Q, K, V, O, dO, LSE, *head, *grads)
        return grads
    n = hp.nonempty_blocks(bm)
    ws = hp.dirty_stored_workspace(Q, K, bm, n)
    fa.flexattn_backward_stored(Q, K, V, O, dO, LSE, *head, *grads, n, ws)
    torch.cuda.synchronize()
    assert hp.ds_written(ws, bm, n)
    return grads


@pytest.mark.parametrize("S,Bk", [(4100, 64), (4224, 128)])
def test_a_key_that_only_the_other_row_lists(S, Bk):
    """Causal: of the first two rows of blocks only the second lists key 200.  A value there that is not finite must not reach
    the first: 0 times infinity is not 0."""
    import paper_2412_05496_amd as fa
    Q, K, V, dO = tensors(2, 16, 16, S, S, S)
    params = fa.ModParams(softcap=30.0)
    bm = fa.alloc_blockmask(1, 1, S, S, 128, Bk, device=DEV)
    fa.flexattn_blockmask_build(fa.MASK_CAUSAL, params, bm)
    print(f"[case] S={S} Bk={Bk}", flush=True)
    want = backward(fa.SCORE_SOFTCAP, fa.MASK_CAUSAL, params, bm, Q, K, V, dO, True)[0][:, :, :128].clone()
    K[:, :, 200, 5] = float("inf")
    got = backward(fa.SCORE_SOFTCAP, fa.MASK_CAUSAL, params, bm, Q, K, V, dO, True)[0][:, :, :128]
    assert torch.isfinite(want.float()).all() and torch.equal(got, want)


@pytest.mark.parametrize("mask,q_len,kv_len,Hq,Bk", [
    ("none", 300, 33000, 345, 64),        # two rows of blocks, and one alone: two segments, the second ragged
    ("causal", 300, 33000, 345, 64),      # the second segment is empty
    ("none", 256, 65700, 513, 128),       # two tiles to a column
    ("none", 130, 33000, 256, 64),        # two heads: 516 tiles
    ("causal", 130, 33000, 256, 64)])
def test_lists_longer_than_a_segment(mask, q_len, kv_len, Hq, Bk):
    """Against the recomputed dQ: the same bf16 dS and K, added up in another order in fp32; one bf16 rounding of each, 2^-8 of the
    larger values."""
    import paper_2412_05496_amd as fa
    Q, K, V, dO = tensors(1, Hq, 1, q_len, kv_len, q_len + Hq)
    params, mask_id = fa.ModParams(), {"none": fa.MASK_NONE, "causal": fa.MASK_CAUSAL}[mask]
    if mask == "causal":                  # (the mask's last keys are hidden from everybody: what dS could hold there is not read)
        K[:, :, 512:] = float("nan")
    bm = fa.alloc_blockmask(1, 1, q_len, kv_len, 128, Bk, device=DEV)
    fa.flexattn_blockmask_build(mask_id, params, bm)
    print(f"[case] {mask} q_len={q_len} kv_len={kv_len} heads={Hq} Bk={Bk}", flush=True)
    want = backward(fa.SCORE_IDENTITY, mask_id, params, bm, Q, K, V, dO, False)
    got = backward(fa.SCORE_IDENTITY, mask_id, params, bm, Q, K, V, dO, True)
    assert torch.equal(got[1], want[1]) and torch.equal(got[2], want[2])
    err = (got[0].float() - want[0].float()).abs()
    assert torch.isfinite(got[0].float()).all() and err.max() <= 2 ** -7 * want[0].float().abs().max()
    assert err.mean() <= 2 ** -9 * want[0].float().abs().mean()
