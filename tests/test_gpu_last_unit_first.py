"""The gradients' kernels take the KV heads of a launch in opposite orders: counts of them around the multiples of eight that the XCDs
share, each head against the same head alone, with dS recomputed and in memory, and query heads divided among workgroups."""
import pytest
import torch

from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("stored", [False, True])
@pytest.mark.parametrize("B,Hkv,G", [(1, 1, 1), (1, 7, 1), (2, 4, 2), (3, 3, 1), (5, 3, 2), (4, 6, 1), (50, 8, 1), (401, 1, 1)])
@pytest.mark.parametrize("D", [64, 128])
def test_heads_stay_apart(D, B, Hkv, G, stored):
    import paper_2412_05496_amd as fa
    S, dev = 200, torch.device("cuda:0")
    g = torch.Generator().manual_seed(B * Hkv + D)
    Q, dO = (torch.randn(B, Hkv * G, S, D, generator=g).to(torch.bfloat16).to(dev) for _ in range(2))
    K, V = (torch.randn(B, Hkv, S, D, generator=g).to(torch.bfloat16).to(dev) for _ in range(2))
    bm = fa.alloc_blockmask(1, 1, S, S, 128, 64, device=dev)
    params = fa.ModParams()
    fa.flexattn_blockmask_build(fa.MASK_CAUSAL, params, bm)
    n = hp.nonempty_blocks(bm)
    print(f"[case] B={B} Hkv={Hkv} G={G} D={D} stored={stored}", flush=True)

    def gradients(Q, K, V, dO):
        O, LSE = torch.empty_like(Q), torch.empty(Q.shape[:3], device=dev)
        head = (fa.SCORE_IDENTITY, fa.MASK_CAUSAL, params, bm, D ** -0.5)
        fa.flexattn_forward(Q, K, V, *head, O, LSE)
        dQ, Vs, _ = hp.dq_and_v_in_one_storage(Q, V)
        out = [dQ, torch.full_like(K, float("nan")), torch.full_like(V, float("nan"))]
        if stored:
            fa.flexattn_backward_stored(Q, K, Vs, O, dO, LSE, *head, *out, n, hp.dirty_stored_workspace(Q, K, bm, n))
        else:
            out[0] = torch.full_like(Q, float("nan"))
            fa.flexattn_backward(Q, K, V, O, dO, LSE, *head, *out)
        return out

    whole = gradients(Q, K, V, dO)
    for b, h in {(0, 0), (B - 1, Hkv - 1), (B // 2, Hkv // 2), ((B - 1) * 7 // 8, 0)}:
        q, kv = slice(h * G, (h + 1) * G), slice(h, h + 1)
        alone = gradients(*(t[b:b + 1, s].contiguous() for t, s in ((Q, q), (K, kv), (V, kv), (dO, q))))
        torch.cuda.synchronize()
        for name, got, want, s in zip(("dQ", "dK", "dV"), whole, alone, (q, kv, kv)):
            got, want = got[b, s].float(), want[0].float()
            # (another kernel may add in another order, in fp32: a bf16 rounding of the larger values)
            assert (got - want).abs().max() <= 2 ** -7 * want.abs().max(), (name, b, h)
