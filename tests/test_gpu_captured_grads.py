"""GPU parity of the gradients of captured tensors (ALiBi bias per head, relative-bias table) against
the oracle, through the C ABI."""
import pytest
import torch

import flex_workloads as wlm
from oracle import flex_oracle as fo
from tests import helpers as hp

pytestmark = pytest.mark.gpu

CASES = [
    ("causal_alibi_d64_gqa", wlm.CFG3, dict(B=2, Hq=4, Hkv=2, S=512, mask="causal")),
    ("doc_alibi_d64", wlm.CFG3, dict(B=2, Hq=4, Hkv=4, S=1024, doc_len_min=60, doc_len_max=500)),
    ("swa_prefix_relbias_gqa_d128", wlm.CFG4, dict(B=2, Hq=4, Hkv=2, S=1024, window=300, prefix_len=100, rel_len=64)),
    ("relbias_d128_bq64_ragged", wlm.CFG4, dict(B=1, Hq=2, Hkv=2, S=1000, Bq=64, window=150, prefix_len=70, rel_len=256)),
    ("causal_alibi_d64_ragged", wlm.CFG3, dict(B=1, Hq=2, Hkv=1, S=333, mask="causal", Bq=64, Bk=128)),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_captured_gradients_match_oracle(case):
    import paper_2412_05496_amd as fa
    name, base, over = case
    dev = torch.device("cuda:0")
    wl = base.scaled(name="captured_" + name, seed=3600 + len(name), **over)
    inp = wlm.make_train_inputs(wl, with_dO=True)
    score_mod, mask_mod = hp.oracle_mods(wl, inp)
    ref = fo.flex_attention_backward_captured(inp.Q, inp.K, inp.V, inp.dO, score_mod, mask_mod, inp.scale)

    O, LSE, bm, (mask_id, score_id, params, Q, K, V) = hp.run_forward(wl, inp, dev)
    dO = inp.dO.to(dev)
    d_alibi = torch.full((wl.Hq,), float("nan"), device=dev) if "alibi_bias" in ref else None
    d_rel = torch.full((wl.Hq, wl.rel_len), float("nan"), device=dev) if "rel_bias" in ref else None
    for _ in range(2):      # written, not accumulated: a second call gives the same
        fa.flexattn_backward_captured(Q, K, V, O, dO, LSE, score_id, mask_id, params, bm, inp.scale, d_alibi, d_rel)
    torch.cuda.synchronize()
    # These sums run over EVERY (q, kv) pair of a head (the ALiBi one weighted by q - kv), so the
    # rounding of delta = rowsum(dO * O) from the bf16 O, which shifts all dS of a row the same way,
    # does not average out as it does in dQ / dK / dV: mean error <= 1e-2 of the mean magnitude.
    if d_alibi is not None:
        hp.check_grad("d_alibi_bias", d_alibi, ref["alibi_bias"], mean_tol=1e-2)
    if d_rel is not None:
        hp.check_grad("d_rel_bias", d_rel, ref["rel_bias"], mean_tol=1e-2)
        assert float(ref["rel_bias"].abs().max()) > 0


@pytest.mark.parametrize("D,S,Bq,rel_len,score,over", [
    (64, 65, 64, 1, "rel_bias", dict(window=10, prefix_len=3)),          # first entry == last entry
    (64, 200, 128, 2, "rel_bias", dict(window=300, prefix_len=150)),     # whole prefix on the first entry
    (128, 131, 128, 33, "rel_bias", dict(window=64, prefix_len=40)),
    (64, 300, 128, 1024, "rel_bias", dict(window=200, prefix_len=10)),   # a table longer than the sequence
    (128, 150, 64, 40, "rel_bias_softcap", dict(mask="doc_causal", doc_len_min=40, doc_len_max=70, softcap=20.0)),
])
def test_captured_diagonals(D, S, Bq, rel_len, score, over):
    """Sums along the diagonals of 32 x 32 blocks: clamped ends, ragged rows, hidden elements."""
    import paper_2412_05496_amd as fa
    dev = torch.device("cuda:0")
    wl = wlm.CFG4.scaled(name="diagonals", B=1, Hq=2, Hkv=1, S=S, D=D, Bq=Bq, rel_len=rel_len, score=score, seed=3700 + S, **over)
    inp = wlm.make_train_inputs(wl, with_dO=True)
    score_mod, mask_mod = hp.oracle_mods(wl, inp)
    ref = fo.flex_attention_backward_captured(inp.Q, inp.K, inp.V, inp.dO, score_mod, mask_mod, inp.scale)
    O, LSE, bm, (mask_id, score_id, params, Q, K, V) = hp.run_forward(wl, inp, dev)
    d_rel = torch.full((wl.Hq, rel_len), float("nan"), device=dev)
    fa.flexattn_backward_captured(Q, K, V, O, inp.dO.to(dev), LSE, score_id, mask_id, params, bm, inp.scale, None, d_rel)
    torch.cuda.synchronize()
    if rel_len == 1:
        # every pair on one entry: the true sum is 0 (P (dP - delta) sums to 0 over a row), what is left is the
        # rounding of O, and of P inside it, to bf16: errors of up to 2^-9 and of random sign on the terms of
        # sum(dO * O), so eight times 2^-9 times their root sum of squares bounds it
        bound = 8 * 2.0 ** -9 * (inp.dO.double() * O.double().cpu()).pow(2).sum(dim=(0, 2, 3)).sqrt()
        assert (d_rel[:, 0].double().cpu().abs() <= bound).all(), (d_rel, bound)
        return
    hp.check_grad("d_rel_bias", d_rel, ref["rel_bias"], mean_tol=1e-2)


def test_score_mods_without_captured_tensors_are_refused():
    import paper_2412_05496_amd as fa
    dev = torch.device("cuda:0")
    wl = wlm.CFG1
    inp = wlm.make_train_inputs(wl, with_dO=True)
    O, LSE, bm, (mask_id, score_id, params, Q, K, V) = hp.run_forward(wl, inp, dev)
    with pytest.raises(fa.FlexAttnError):
        fa.flexattn_backward_captured(Q, K, V, O, inp.dO.to(dev), LSE, score_id, mask_id, params, bm, inp.scale)
