"""Every (batch entry, KV head) and every row and column of blocks is computed, whatever their number: workgroups are
dealt to the XCDs eight (batch, KV head) units at a time and the units that are left in eighths."""
import pytest
import torch

import flex_workloads as wlm
from oracle import flex_oracle as fo
from tests import helpers as hp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hkv,G,S,D", [
    (1, 1, 1, 65, 64), (1, 1, 1, 1100, 128), (1, 2, 3, 300, 64), (3, 1, 2, 640, 64), (1, 5, 1, 130, 128), (3, 2, 1, 577, 64),
    (7, 1, 1, 520, 64), (1, 8, 1, 200, 64), (3, 3, 1, 450, 64), (5, 2, 2, 140, 128), (1, 15, 1, 260, 64), (17, 1, 1, 330, 64)])
def test_every_unit_and_piece(B, Hkv, G, S, D):
    import paper_2412_05496_amd as fa
    dev = torch.device("cuda:0")
    wl = wlm.CFG3.scaled(name="units", B=B, Hq=Hkv * G, Hkv=Hkv, S=S, D=D, mask="causal", Bq=64 if S < 400 else 128, Bk=64, seed=7100 + B * Hkv)
    inp = wlm.make_train_inputs(wl, with_dO=True)
    score_mod, mask_mod = hp.oracle_mods(wl, inp)
    O_ref, LSE_ref = fo.flex_attention(inp.Q, inp.K, inp.V, score_mod, mask_mod, inp.scale)
    ref = fo.flex_attention_backward(inp.Q, inp.K, inp.V, inp.dO, score_mod, mask_mod, inp.scale)
    O, LSE, bm, ids = hp.run_forward(wl, inp, dev)
    hp.check_output(O, LSE, O_ref, LSE_ref)
    for stored in (False, True):
        for name, got, want in zip(("dQ", "dK", "dV"), hp.run_backward(wl, inp, dev, O, LSE, bm, ids, stored=stored), ref):
            hp.check_grad(name, got, want)
    # the captured sums of all batch entries at once against those of one entry after the other.  A workgroup adds the sums
    # of up to four waves in any order; they are below 1e3 here, so that a workgroup may differ by 2 * 2^-24 * 1e3.
    mask_id, score_id, params, Q, K, V = ids
    dO = inp.dO.to(dev)

    def captured(b):
        d = torch.full((wl.Hq,), float("nan"), device=dev)
        fa.flexattn_backward_captured(Q[b], K[b], V[b], O[b], dO[b], LSE[b].contiguous(), score_id, mask_id, params, bm, inp.scale, d, None)
        return d.double()
    got, want = captured(slice(0, B)), sum(captured(slice(b, b + 1)) for b in range(B))
    assert float((got - want).abs().max()) <= 1.2e-4 * B * -(-S // wl.Bq) + 1e-6 * float(want.abs().max())
