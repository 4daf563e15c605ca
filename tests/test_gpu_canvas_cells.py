"""Canvases whose 32 consecutive tokens are cells of 8 x 4 pixels (tiles of 8 x 8, Morton order), in kernels of their own: windows
up to the widest that their 64 columns and lines hold and the next one, which is compared as other canvases are; forward and
gradients against the oracle, and against the general kernels (offsets, all 0, take a call there)."""
import pytest
import torch

from oracle import flex_oracle as fo
from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("W,H,K,layout,Bq,Bk", [
    (8, 8, 7, "morton", 128, 64), (8, 24, 3, "tiled", 64, 128),             # one cell wide; half of a last block of queries is no pixel
    (16, 16, 9, "morton", 64, 64), (32, 32, 29, "morton", 128, 64),         # keys that reach both borders: up to r = 14
    (32, 32, 31, "morton", 128, 128), (64, 64, 33, "morton", 128, 64),      # r = 15, 16 there: not cells
    (64, 64, 27, "morton", 64, 128), (64, 56, 29, "tiled", 128, 64),
    (24, 104, 15, "tiled", 64, 64), (104, 24, 23, "tiled", 128, 64),
    (80, 80, 33, "tiled", 128, 128)])                                       # r = 16, one border at a time
def test_cells(W, H, K, layout, Bq, Bk, D):
    import paper_2412_05496_amd as fa
    dev = torch.device("cuda:0")
    S = W * H
    g = torch.Generator().manual_seed(S * K + D)
    Q, dO = (torch.randn(1, 2, S, D, generator=g).to(torch.bfloat16).float() for _ in range(2))
    Kt, V = (torch.randn(1, 1, S, D, generator=g).to(torch.bfloat16).float() for _ in range(2))
    mask = fo.neighborhood_mask(W, H, K, layout, 8)
    O_ref, LSE_ref = fo.flex_attention(Q, Kt, V, fo.Identity(), mask, D ** -0.5)
    refs = fo.flex_attention_backward(Q, Kt, V, dO, fo.Identity(), mask, D ** -0.5)
    params = fa.ModParams(na_width=W, na_height=H, na_kernel=K, na_layout={"tiled": fa.NA_TILED, "morton": fa.NA_MORTON}[layout],
                          na_tile=8 if layout == "tiled" else 0)
    bm = fa.alloc_blockmask(1, 1, S, S, Bq, Bk, device=dev)
    fa.flexattn_blockmask_build(fa.MASK_NEIGHBORHOOD, params, bm)
    n = hp.nonempty_blocks(bm)
    print(f"[case] {W} x {H} K={K} {layout} {Bq} x {Bk} D={D}", flush=True)
    for copies in (1, max(1, 400000 // S)):                 # few workgroups and many
        q, k, v, do = (t.to(torch.bfloat16).to(dev).expand(copies, -1, -1, -1) for t in (Q, Kt, V, dO))
        both = []
        for offsets in (None, torch.zeros(copies, dtype=torch.int32, device=dev)):
            params.q_offsets = offsets
            head = (fa.SCORE_IDENTITY, fa.MASK_NEIGHBORHOOD, params, bm, D ** -0.5)
            O, LSE = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device=dev), torch.full(q.shape[:3], float("nan"), device=dev)
            fa.flexattn_forward(q, k, v, *head, O, LSE)
            grads = [torch.full(t.shape, float("nan"), dtype=torch.bfloat16, device=dev) for t in (q, k, v)]
            fa.flexattn_backward(q, k, v, O, do, LSE, *head, *grads)
            ws = torch.full((fa.flexattn_backward_stored_workspace_bytes(q, k, bm, n),), 0xFF, dtype=torch.uint8, device=dev)
            stored = [torch.full(t.shape, float("nan"), dtype=torch.bfloat16, device=dev) for t in (q, k, v)]
            fa.flexattn_backward_stored(q, k, v, O, do, LSE, *head, *stored, n, ws)
            torch.cuda.synchronize()
            hp.check_output(O[:1], LSE[:1], O_ref, LSE_ref)
            for got in (grads, stored):
                for name, t, ref in zip(("dQ", "dK", "dV"), got, refs):
                    hp.check_grad(name, t[:1], ref)
                    assert torch.equal(t, t[:1].expand_as(t)), name
            both.append((O, LSE, *grads, *stored))
        # the same sums over the same elements; exp2's argument, where a row's maximum is an older one, may differ in its last bits
        for cells, general in zip(*both):
            err = (cells.float() - general.float()).abs().max()
            assert err <= 2 ** -7 * general.float().abs().max(), err
