"""The forward at D = 64 with rows of blocks of 128 on long rows without a window: its tile pipeline with a tracked maximum, which
is taken by the number of workgroups (8 units at a time, see unit_grid: 20, 31 and 34 copies of 32 rows of blocks are 640, 992 and 1088
of them; 36 of 33 1216, 68 of 17 1184), and the plain form on the other side of each line.  Copies share their inputs and must agree bit
for bit; O and LSE against the oracle at the tolerances of tests/helpers.py."""
import math

import pytest
import torch

from oracle import flex_oracle as fo
from tests import helpers as hp
from tests.test_gpu_running_maximum import STEPS

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def check(Q, K, V, score_id, score, mask_id, mask, params, scale, Bk, copies):
    import paper_2412_05496_amd as fa
    O_ref, LSE_ref = fo.flex_attention(Q, K, V, score, mask, scale)
    bm = fa.alloc_blockmask(1, 1, Q.shape[2], K.shape[2], 128, Bk, device=DEV)
    fa.flexattn_blockmask_build(mask_id, params, bm)
    for n in copies:
        q, k, v = (t.to(torch.bfloat16).to(DEV).expand(n, -1, -1, -1) for t in (Q, K, V))
        O = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device=DEV)
        LSE = torch.full(q.shape[:3], float("nan"), device=DEV)
        print(f"  {n} copies", flush=True)
        fa.flexattn_forward(q, k, v, score_id, mask_id, params, bm, scale, O, LSE)
        torch.cuda.synchronize()
        assert torch.equal(O, O[:1].expand_as(O)) and torch.equal(LSE, LSE[:1].expand_as(LSE))
        # (LSE in fp32 is exact to 2^-24 of its size: 5e-5 at 700)
        hp.check_output(O[:1], LSE[:1], O_ref, LSE_ref)


def randn(seed, q_len, kv_len):
    gen = torch.Generator().manual_seed(seed)
    return [torch.randn(1, 1, n, 64, generator=gen).to(torch.bfloat16).float() for n in (q_len, kv_len, kv_len)]


@pytest.mark.parametrize("mask,score,q_len,kv_len,Bk,copies", [
    ("none", "identity", 4090, 4100, 64, (20, 31, 34)), ("none", "identity", 4096, 4096, 128, (20, 31, 34)), ("none", "identity", 4096, 4095, 64, (20,)),
    ("causal", "identity", 4100, 4100, 64, (36, 48)), ("causal", "identity", 4224, 4224, 128, (36,)), ("prefix_lm", "identity", 4100, 4100, 64, (36,)),
    ("causal", "alibi-", 4100, 4100, 64, (36, 48)), ("causal", "alibi+", 4100, 4100, 64, (36, 48)), ("causal", "alibi-", 4130, 4130, 128, (36,)),
    ("causal", "softcap", 2050, 2050, 64, (68,)), ("causal", "softcap", 2176, 2176, 128, (68,)), ("causal", "softcap", 2040, 2047, 64, (70,)),
    ("causal", "alibi_softcap-", 2050, 2050, 64, (68,)), ("causal", "alibi_softcap+", 2050, 2050, 64, (68,))])
def test_either_side_of_the_lines(mask, score, q_len, kv_len, Bk, copies):
    import paper_2412_05496_amd as fa
    print(f"[case] {mask} {score} q_len={q_len} kv_len={kv_len} Bk={Bk}", flush=True)
    params = fa.ModParams(softcap=60.0, prefix_len=100)
    params.alibi_bias = torch.tensor([0.004 if score[-1] == "+" else -0.02], dtype=torch.float32, device=DEV)
    bias = params.alibi_bias.double().cpu()
    score_id, mod = {"identity": (fa.SCORE_IDENTITY, fo.Identity()), "softcap": (fa.SCORE_SOFTCAP, fo.Softcap(60.0)),
                     "alibi": (fa.SCORE_ALIBI, fo.Alibi(bias)),
                     "alibi_softcap": (fa.SCORE_ALIBI | fa.SCORE_SOFTCAP, fo.Compose(fo.Alibi(bias), fo.Softcap(60.0)))}[score.rstrip("-+")]
    mask_id, mask_mod = {"none": (fa.MASK_NONE, fo.no_mask), "causal": (fa.MASK_CAUSAL, fo.causal_mask),
                         "prefix_lm": (fa.MASK_PREFIX_LM, fo.or_mask(fo.causal_mask, fo.prefix_mask(100)))}[mask]
    check(*randn(q_len + Bk, q_len, kv_len), score_id, mod, mask_id, mask_mod, params, 0.125, Bk, copies)


@pytest.mark.parametrize("steps", sorted(STEPS))
@pytest.mark.parametrize("mask,copies", [("none", 20), ("causal", 36)])
def test_maxima_that_move(steps, mask, copies):
    import paper_2412_05496_amd as fa
    S = 4100
    print(f"[case] {steps} {mask}", flush=True)
    Q, K, V = randn(97, S, S)
    Q.zero_(), K.zero_()
    Q[..., 0] = 1.0
    Q[:, :, ::3, 0] = -0.5                  # (rows of one wave whose maxima move at different blocks)
    K[..., 0] = torch.tensor(STEPS[steps]).repeat_interleave(32).repeat(S // 320 + 1)[:S].to(torch.bfloat16).float()
    mask_id, mask_mod = {"none": (fa.MASK_NONE, fo.no_mask), "causal": (fa.MASK_CAUSAL, fo.causal_mask)}[mask]
    check(Q, K, V, fa.SCORE_IDENTITY, fo.Identity(), mask_id, mask_mod, fa.ModParams(), math.log(2.0), 64, (copies,))
