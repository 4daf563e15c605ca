"""D = 128 gradients of neighborhood masks whose columns of blocks list more steps than the dK/dV kernel lays
out at once: more than 64 (a wave's chunk) and more than 512 (a segment), with steps and blocks that are left out
at the start, in the middle and at the end of both."""
import pytest
import torch

import flex_workloads as wlm
from oracle import flex_oracle as fo
from tests import helpers as hp

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def canvas(fa, w, h, k, layout, tile):
    return fa.ModParams(na_width=w, na_height=h, na_kernel=k, na_tile=tile,
                        na_layout={"row_major": fa.NA_ROW_MAJOR, "tiled": fa.NA_TILED, "morton": fa.NA_MORTON}[layout])


def forward(fa, inp, params, Bq, Bk):
    S = inp.Q.shape[2]
    bm = fa.alloc_blockmask(1, 1, S, S, Bq, Bk, device=DEV)
    fa.flexattn_blockmask_build(fa.MASK_NEIGHBORHOOD, params, bm)
    Q, K, V = (t.to(DEV) for t in (inp.Q, inp.K, inp.V))
    O, LSE = torch.full_like(Q, float("nan")), torch.full(Q.shape[:3], float("nan"), device=DEV)
    fa.flexattn_forward(Q, K, V, fa.SCORE_IDENTITY, fa.MASK_NEIGHBORHOOD, params, bm, inp.scale, O, LSE)
    torch.cuda.synchronize()
    return O, LSE, bm, (fa.MASK_NEIGHBORHOOD, fa.SCORE_IDENTITY, params, Q, K, V)


@pytest.mark.parametrize("w,h,k,layout,tile,Bq,Bk", [(128, 40, 39, "row_major", 0, 128, 64), (128, 40, 39, "row_major", 0, 64, 128),
                                                     (72, 72, 59, "tiled", 8, 128, 64), (72, 72, 45, "tiled", 8, 128, 128)])
def test_more_than_64_steps(w, h, k, layout, tile, Bq, Bk):
    import paper_2412_05496_amd as fa
    S = w * h
    wl = wlm.CFG2.scaled(name="canvas64", B=1, Hq=2, Hkv=1, S=S, Bq=Bq, Bk=Bk, mask="none", score="identity", seed=5100 + S)
    inp = wlm.make_train_inputs(wl, with_dO=True)
    mask_mod = fo.neighborhood_mask(w, h, k, layout, tile)
    print(f"[case] canvas {w}x{h} K={k} {layout} blocks {Bq}x{Bk}", flush=True)
    O, LSE, bm, ids = forward(fa, inp, canvas(fa, w, h, k, layout, tile), Bq, Bk)
    assert int((bm.q_num_blocks + bm.full_q_num_blocks).max()) * (Bq // 64) > 64
    hp.check_output(O, LSE, *fo.flex_attention(inp.Q, inp.K, inp.V, fo.Identity(), mask_mod, inp.scale))
    ref = fo.flex_attention_backward(inp.Q, inp.K, inp.V, inp.dO, fo.Identity(), mask_mod, inp.scale)
    for stored in (False, True):
        for name, got, r in zip(("dQ", "dK", "dV"), hp.run_backward(wl, inp, torch.device(DEV), O, LSE, bm, ids, stored=stored), ref):
            hp.check_grad(name, got, r)


@pytest.mark.parametrize("layout,tile", [("row_major", 0), ("tiled", 8)])
def test_more_than_512_steps(layout, tile):
    """256 x 256 pixels, K = 201: about 800 steps per column.  Output and gradients of 192 tokens (the first, middle
    and last 64) against the definition in 64 bits."""
    import paper_2412_05496_amd as fa
    w = h = 256
    k, S = 201, w * h
    wl = wlm.CFG2.scaled(name="canvas512", B=1, Hq=1, Hkv=1, S=S, Bq=128, Bk=64, mask="none", score="identity", seed=5200)
    inp = wlm.make_train_inputs(wl, with_dO=True)
    mask_mod = fo.neighborhood_mask(w, h, k, layout, tile)
    print(f"[case] canvas {w}x{h} K={k} {layout}", flush=True)
    O, LSE, bm, ids = forward(fa, inp, canvas(fa, w, h, k, layout, tile), 128, 64)
    assert int((bm.q_num_blocks + bm.full_q_num_blocks).max()) * 2 > 512

    at = torch.cat([torch.arange(64), S // 2 - 1000 + torch.arange(64), S - 64 + torch.arange(64)])
    every = torch.arange(S)
    Q, K, V, dO = (t[0, 0].double() for t in (inp.Q, inp.K, inp.V, inp.dO))
    O_all, LSE_all = O[0, 0].double().cpu(), LSE[0, 0].double().cpu()
    delta = (dO * O_all).sum(1, keepdim=True)
    O_ref, LSE_ref = fo.attention_head(Q, K, V, fo.Identity(), mask_mod, inp.scale, 0, 0, at)
    hp.check_output(O[:, :, at], LSE[:, :, at], O_ref[None, None], LSE_ref[None, None])

    def p_and_ds(rows, cols):
        P = torch.exp(inp.scale * (Q[rows] @ K[cols].T) - LSE_all[rows, None])
        P = torch.where(mask_mod(0, 0, rows.view(-1, 1), cols.view(1, -1)), P, torch.zeros_like(P))
        return P, P * (dO[rows] @ V[cols].T - delta[rows])
    P, dS = p_and_ds(every, at)
    dV_ref, dK_ref = P.T @ dO, inp.scale * (dS.T @ Q)
    dQ_ref = inp.scale * (p_and_ds(at, every)[1] @ K)
    for stored in (False, True):
        dQ, dK, dV = hp.run_backward(wl, inp, torch.device(DEV), O, LSE, bm, ids, stored=stored)
        for name, got, ref in (("dQ", dQ, dQ_ref), ("dK", dK, dK_ref), ("dV", dV, dV_ref)):
            hp.check_grad(name, got[0, 0, at], ref)
            assert torch.isfinite(got.float()).all()
