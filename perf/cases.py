"""Performance cases of the FlexAttention path: the calls a training step, a prompt and a decoding loop make.

    listed()  the named cases            draw(rng)    one more case of the same ranges
    prepare(case, seed)  what the caller holds before the call, on the GPU
    run(state)           one pass through the public entry points, and its outputs
    work(case)           bytes and operations the pass cannot do without
    tolerance(case)      how far two correct implementations at the same precision may be apart

Three kinds of call:
    train    (BlockMask build where the mask follows the batch,) forward, backward; "forward" is its
             first half (evaluation, an encoder)
    prefill  a chunk of new tokens per sequence on top of a paged cache: BlockMask build for the
             chunk's positions, conversion of its lists to pool pages, paged forward
    decode   one new token per sequence against a paged cache
"""
import math
import random

import torch

import paper_2412_05496_amd as fa

MASKS = {"none": fa.MASK_NONE, "causal": fa.MASK_CAUSAL, "window": fa.MASK_SWA_CAUSAL, "prefix": fa.MASK_PREFIX_LM,
         "documents": fa.MASK_DOCUMENT_CAUSAL, "window_or_prefix": fa.MASK_SWA_CAUSAL_OR_PREFIX,
         "neighborhood": fa.MASK_NEIGHBORHOOD}
SCORES = {"identity": fa.SCORE_IDENTITY, "alibi": fa.SCORE_ALIBI, "softcap": fa.SCORE_SOFTCAP,
          "rel_bias": fa.SCORE_REL_BIAS, "alibi_softcap": fa.SCORE_ALIBI | fa.SCORE_SOFTCAP,
          "rel_bias_softcap": fa.SCORE_REL_BIAS | fa.SCORE_SOFTCAP}
LAYOUTS = {"row_major": fa.NA_ROW_MAJOR, "tiled": fa.NA_TILED, "morton": fa.NA_MORTON}
# the (mask_mod, score_mod) pairs forward and backward are compiled for
PAIRS = [("none", "identity"), ("causal", "identity"), ("causal", "alibi"), ("causal", "softcap"),
         ("window", "identity"), ("prefix", "identity"), ("documents", "identity"), ("documents", "alibi"),
         ("window_or_prefix", "rel_bias"), ("neighborhood", "identity"), ("window", "softcap"),
         ("causal", "alibi_softcap"), ("documents", "rel_bias_softcap")]


def train(name, B, Hq, Hkv, S, D, mask, score="identity", backward="recompute", **kw):
    """backward: "none", "recompute" (flexattn_backward) or "stored" (flexattn_backward_stored);
    rebuild: the mask follows the batch's data, so the step builds its BlockMask;
    captured: the step also trains the score_mod's tensor (ALiBi bias, relative-bias table)."""
    case = dict(kind="train", name=name, B=B, Hq=Hq, Hkv=Hkv, S=S, D=D, Bq=128, Bk=64, mask=mask, score=score,
                backward=backward, rebuild=False, captured=False, window=0, prefix_len=0, softcap=30.0, rel_len=256,
                doc_min=256, doc_max=4096, width=0, height=0, kernel=0, layout="row_major", tile=0)
    case.update(kw)
    return case


def prefill(name, nseq, Hq, Hkv, D, chunk, cached_min, cached_max, page, score="identity"):
    return dict(kind="prefill", name=name, nseq=nseq, Hq=Hq, Hkv=Hkv, D=D, chunk=chunk, cached_min=cached_min,
                cached_max=cached_max, page=page, score=score, softcap=30.0)


def decode(name, nseq, Hq, Hkv, D, ctx_min, ctx_max, page, score="identity", window=-1):
    return dict(kind="decode", name=name, nseq=nseq, Hq=Hq, Hkv=Hkv, D=D, ctx_min=ctx_min, ctx_max=ctx_max, page=page,
                score=score, window=window, softcap=30.0, rel_len=256)


def listed():
    return [
        # a short prompt through a small causal model, no gradients: launches and latency
        train("forward_small", 1, 2, 2, 256, 64, "causal", backward="none", Bq=64),
        # an encoder without a mask on a length that fits no block
        train("forward_encoder_ragged", 8, 16, 16, 777, 64, "none", backward="none"),
        # serving, long prompts: 2048 new tokens per sequence on top of a cache of up to 16k
        prefill("prefill_chunk", 4, 32, 8, 128, 2048, 4096, 14336, 64),
        # serving, one user: the next token of one sequence
        decode("decode_one", 1, 32, 8, 128, 7000, 8192, 16),
        # serving, a small model: short contexts, ALiBi, larger pages
        decode("decode_short_alibi", 16, 16, 4, 64, 100, 4096, 64, score="alibi"),
        # serving, a full batch of 64 sequences with contexts of 1k to 32k tokens
        decode("decode_batch_ragged", 64, 32, 8, 128, 1024, 32768, 16),
        # training on many short sequences
        train("train_short", 64, 16, 16, 1024, 64, "causal"),
        # training, long sliding window with grouped heads, a length that fits no block
        train("train_window_gqa", 4, 16, 2, 5000, 64, "window", window=1024),
        # training on packed documents: the BlockMask is built from each batch's document ids
        train("train_documents", 1, 16, 16, 16384, 64, "documents", "alibi", rebuild=True),
        # training on images: 128 x 128 pixels, each attends to the 13 x 13 pixels around it
        train("train_neighborhood", 4, 16, 16, 16384, 64, "neighborhood", backward="stored", width=128, height=128,
              kernel=13, layout="tiled", tile=8),
        # the headline training step: dense causal attention with a tanh soft-cap
        train("train_softcap", 4, 16, 16, 8192, 128, "causal", "softcap", backward="stored", rebuild=True),
        # long context, grouped heads, a trained relative bias inside a window or a prefix
        train("train_relative_bias", 2, 32, 8, 32768, 128, "window_or_prefix", "rel_bias", backward="stored",
              captured=True, window=4096, prefix_len=1024),
    ]


# ---- more cases of the same ranges -------------------------------------------------------------
MOST_FLOPS = 1.5e13       # of the largest listed case: 1.78e13


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _heads(rng, most):
    hkv = rng.choice([h for h in (1, 2, 4, 8, 16) if h <= most])
    return hkv * rng.choice([g for g in (1, 1, 2, 4, 8) if hkv * g <= most]), hkv


def _draw_train(rng):
    mask, score = rng.choice(PAIRS)
    D = rng.choice([64, 128])
    Hq, Hkv = _heads(rng, 32)
    kw = dict(Bq=rng.choice([128, 128, 64]), Bk=rng.choice([64, 64, 128]),
              backward=rng.choice(["none", "recompute", "recompute", "stored"]), rebuild=mask == "documents")
    S = _log(rng, 200, 32768)
    if mask == "neighborhood":
        layout = rng.choice(sorted(LAYOUTS))
        if layout == "morton":
            w = h = rng.choice([16, 32, 64, 128])
        elif layout == "tiled":
            w, h = 8 * rng.randint(2, 16), 8 * rng.randint(2, 16)
        else:
            w, h = rng.randint(15, 128), rng.randint(15, 128)
        S = w * h
        kw.update(width=w, height=h, kernel=2 * rng.randint(1, min(13, (min(w, h) - 1) // 2)) + 1, layout=layout,
                  tile=8 if layout == "tiled" else 0)
    if "window" in mask:
        kw["window"] = _log(rng, 64, 4096)
    if "prefix" in mask:
        kw["prefix_len"] = rng.randint(1, max(1, S // 4))
    if mask == "documents" and kw["backward"] == "stored":
        kw["backward"] = "recompute"      # the block count of a mask built in the step is not known on the host
    if "rel_bias" in score:
        kw["rel_len"] = rng.randint(16, 512)
    kw["captured"] = kw["backward"] != "none" and ("alibi" in score or "rel_bias" in score) and rng.random() < 0.5
    case = train("", 1, Hq, Hkv, S, D, mask, score, **kw)
    # as many sequences as fit the step: up to 64k tokens, no more work or memory than the listed cases
    most = max(1, min(64, 65536 // S))
    one = work(case)["flops"]
    most = max(1, min(most, int(MOST_FLOPS / one)))
    if kw["backward"] == "stored":        # two bytes per score inside a visited block; 3 are allowed for
        most = max(1, min(most, int(2e10 / (3.0 * S * S * Hq))))
    case["B"] = _log(rng, 1, most)
    if one > MOST_FLOPS or (kw["backward"] == "stored" and 3.0 * S * S * Hq > 2e10):
        return None
    return case


def _draw_prefill(rng):
    page, D = rng.choice([64, 128]), rng.choice([64, 128])
    Hq, Hkv = _heads(rng, 32)
    chunk = _log(rng, 64, 4096)
    lo = rng.randint(0, 4096)
    return prefill("", rng.randint(1, 8), Hq, Hkv, D, chunk, lo, lo + _log(rng, 64, 16384), page,
                   rng.choice(["identity", "identity", "alibi", "softcap"]))


def _draw_decode(rng):
    D = rng.choice([64, 128, 128])
    Hq, Hkv = _heads(rng, 32)
    score = rng.choice(["identity", "identity", "alibi", "softcap", "rel_bias"])
    ctx_max = _log(rng, 128, 65536)
    nseq = _log(rng, 1, max(1, min(256, 1500000 // ctx_max)))
    return decode("", nseq, Hq, Hkv, D, rng.randint(1, ctx_max), ctx_max, rng.choice([16, 16, 32, 64, 128]), score,
                  _log(rng, 64, 4096) if rng.random() < 0.2 else -1)


def draw(rng):
    while True:
        case = rng.choice([_draw_train, _draw_train, _draw_prefill, _draw_decode, _draw_decode])(rng)
        if case is not None and work(case)["flops"] <= MOST_FLOPS:
            del case["name"]
            return case


# ---- inputs ----------------------------------------------------------------------------------------
def _document_lengths(rng, S, lo, hi):
    out = []
    while S > 0:
        out.append(min(rng.randint(lo, hi), S))
        S -= out[-1]
    return out


def _randn(gen, *shape):
    return torch.randn(*shape, generator=gen, dtype=torch.bfloat16, device="cuda")


def _mods(case, gen):
    """The tensors the score_mod captures."""
    p = fa.ModParams(softcap=case["softcap"])
    if "alibi" in case["score"]:
        H = case["Hq"]
        p.alibi_bias = torch.tensor([-2.0 ** (-8.0 * (h + 1) / H) for h in range(H)], dtype=torch.float32).cuda()
    if "rel_bias" in case["score"]:
        p.rel_bias = 0.1 * torch.randn(case["Hq"], case["rel_len"], generator=gen, dtype=torch.float32, device="cuda")
    return p


def _prepare_train(case, rng, gen):
    B, Hq, Hkv, S, D = (case[k] for k in ("B", "Hq", "Hkv", "S", "D"))
    s = dict(case=case, mask=MASKS[case["mask"]], score=SCORES[case["score"]], scale=1.0 / math.sqrt(D))
    s["Q"], s["K"], s["V"] = _randn(gen, B, Hq, S, D), _randn(gen, B, Hkv, S, D), _randn(gen, B, Hkv, S, D)
    p = s["params"] = _mods(case, gen)
    p.window, p.prefix_len = case["window"], case["prefix_len"]
    Bm = 1
    if case["mask"] == "documents":
        Bm = B
        ids = []
        for _ in range(B):
            lengths = _document_lengths(rng, S, case["doc_min"], case["doc_max"])
            ids.append(torch.repeat_interleave(torch.arange(len(lengths), dtype=torch.int32), torch.tensor(lengths)))
        p.doc_ids = torch.stack(ids).cuda()
    if case["mask"] == "neighborhood":
        p.na_width, p.na_height, p.na_kernel = case["width"], case["height"], case["kernel"]
        p.na_layout, p.na_tile = LAYOUTS[case["layout"]], case["tile"]
    bm = s["bm"] = fa.alloc_blockmask(Bm, 1, S, S, case["Bq"], case["Bk"])
    s["bm_ws"] = torch.empty(fa.flexattn_blockmask_workspace_bytes(Bm, 1, S, S, case["Bq"], case["Bk"]),
                             dtype=torch.uint8, device="cuda")
    fa.flexattn_blockmask_build(s["mask"], p, bm, s["bm_ws"])
    s["O"] = torch.empty_like(s["Q"])
    s["LSE"] = torch.empty(B, Hq, S, dtype=torch.float32, device="cuda")
    if case["backward"] == "none":
        return s
    s["dO"] = _randn(gen, B, Hq, S, D)
    s["dQ"], s["dK"], s["dV"] = torch.empty_like(s["Q"]), torch.empty_like(s["K"]), torch.empty_like(s["V"])
    if case["backward"] == "stored":
        s["n_blocks"] = int(bm.stats[:2].sum())
        n = fa.flexattn_backward_stored_workspace_bytes(s["Q"], s["K"], bm, s["n_blocks"])
    else:
        n = fa.flexattn_backward_workspace_bytes(s["Q"], s["K"])
    s["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda")
    s["d_alibi"] = s["d_rel"] = None
    if case["captured"] and p.alibi_bias is not None:
        s["d_alibi"] = torch.empty_like(p.alibi_bias)
    if case["captured"] and p.rel_bias is not None:
        s["d_rel"] = torch.empty_like(p.rel_bias)
    return s


def _prepare_cache(case, gen, lengths, longest):
    """A pool whose pages belong to the sequences in random order, and their page table, which has room
    for the longest sequence the server admits."""
    page, Hkv, D = case["page"], case["Hkv"], case["D"]
    counts = [(n + page - 1) // page for n in lengths]
    n_pool = sum(counts)
    order = torch.randperm(n_pool, generator=gen, device="cuda").to(torch.int32)
    table = torch.zeros(len(lengths), (longest + page - 1) // page, dtype=torch.int32, device="cuda")
    at = 0
    for b, n in enumerate(counts):
        table[b, :n] = order[at:at + n]
        at += n
    return _randn(gen, n_pool, Hkv, page, D), _randn(gen, n_pool, Hkv, page, D), table


def _prepare_prefill(case, rng, gen):
    nseq, Hq, D, chunk, page = (case[k] for k in ("nseq", "Hq", "D", "chunk", "page"))
    cached = [rng.randint(case["cached_min"], case["cached_max"]) for _ in range(nseq)]
    s = dict(case=case, score=SCORES[case["score"]], scale=1.0 / math.sqrt(D), params=_mods(case, gen))
    s["Kp"], s["Vp"], s["table"] = _prepare_cache(case, gen, [n + chunk for n in cached], case["cached_max"] + chunk)
    s["params"].q_offsets = torch.tensor(cached, dtype=torch.int32).cuda()
    s["Q"] = _randn(gen, nseq, Hq, chunk, D)
    s["O"] = torch.empty_like(s["Q"])
    s["LSE"] = torch.empty(nseq, Hq, chunk, dtype=torch.float32, device="cuda")
    kv_len = s["table"].shape[1] * page
    bm = s["bm"] = fa.alloc_blockmask(nseq, 1, chunk, kv_len, 128, page)
    s["bm_ws"] = torch.empty(fa.flexattn_blockmask_workspace_bytes(nseq, 1, chunk, kv_len, 128, page),
                             dtype=torch.uint8, device="cuda")
    s["phys"], s["phys_full"] = torch.empty_like(bm.kv_indices), torch.empty_like(bm.full_kv_indices)
    return s


def _prepare_decode(case, rng, gen):
    nseq, Hq, D = case["nseq"], case["Hq"], case["D"]
    ctx = [rng.randint(case["ctx_min"], case["ctx_max"]) for _ in range(nseq)]
    s = dict(case=case, score=SCORES[case["score"]], scale=1.0 / math.sqrt(D), params=_mods(case, gen))
    s["params"].window = max(case["window"], 0)
    s["mask"] = fa.MASK_CTX_LEN if case["window"] < 0 else fa.MASK_CTX_LEN_WINDOW
    s["Kp"], s["Vp"], s["table"] = _prepare_cache(case, gen, ctx, case["ctx_max"])
    s["ctx"] = torch.tensor(ctx, dtype=torch.int32).cuda()
    s["Q"] = _randn(gen, nseq, Hq, D)
    s["O"] = torch.empty(nseq, Hq, D, dtype=torch.bfloat16, device="cuda")
    s["LSE"] = torch.empty(nseq, Hq, dtype=torch.float32, device="cuda")
    s["ws"] = torch.empty(max(16, fa.flexattn_paged_decode_workspace_bytes(s["Q"], s["Kp"], s["table"])),
                          dtype=torch.uint8, device="cuda")
    return s


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    make = {"train": _prepare_train, "prefill": _prepare_prefill, "decode": _prepare_decode}[case["kind"]]
    return make(case, random.Random(seed), gen)


# ---- one pass ---------------------------------------------------------------------------------------
def _run_train(s):
    case, p, bm = s["case"], s["params"], s["bm"]
    if case["rebuild"]:
        fa.flexattn_blockmask_build(s["mask"], p, bm, s["bm_ws"])
    fa.flexattn_forward(s["Q"], s["K"], s["V"], s["score"], s["mask"], p, bm, s["scale"], s["O"], s["LSE"])
    out = {"O": s["O"], "LSE": s["LSE"]}
    if case["rebuild"]:
        out["blocks"] = [bm.kv_num_blocks, bm.kv_indices, bm.full_kv_num_blocks, bm.full_kv_indices, bm.q_num_blocks,
                         bm.q_indices, bm.full_q_num_blocks, bm.full_q_indices, bm.kv_order, bm.q_order, bm.stats]
    if case["backward"] == "none":
        return out
    args = (s["Q"], s["K"], s["V"], s["O"], s["dO"], s["LSE"], s["score"], s["mask"], p, bm, s["scale"])
    if case["backward"] == "stored":
        fa.flexattn_backward_stored(*args, s["dQ"], s["dK"], s["dV"], s["n_blocks"], s["ws"])
    else:
        fa.flexattn_backward(*args, s["dQ"], s["dK"], s["dV"], s["ws"])
    out.update(dQ=s["dQ"], dK=s["dK"], dV=s["dV"])
    if case["captured"]:
        fa.flexattn_backward_captured(*args, s["d_alibi"], s["d_rel"])
        out.update(d_alibi=s["d_alibi"], d_rel=s["d_rel"])
    return out


def _run_prefill(s):
    p, bm = s["params"], s["bm"]
    fa.flexattn_blockmask_build(fa.MASK_CAUSAL, p, bm, s["bm_ws"])
    fa.flexattn_paged_convert_blockmask(bm.kv_num_blocks, bm.kv_indices, s["table"], s["phys"])
    fa.flexattn_paged_convert_blockmask(bm.full_kv_num_blocks, bm.full_kv_indices, s["table"], s["phys_full"])
    fa.flexattn_paged_forward(s["Q"], s["Kp"], s["Vp"], s["score"], fa.MASK_CAUSAL, p, bm, s["phys"], s["phys_full"],
                              s["scale"], s["O"], s["LSE"])
    return {"O": s["O"], "LSE": s["LSE"], "blocks": [bm.kv_num_blocks, bm.full_kv_num_blocks, s["phys"], s["phys_full"]]}


def _run_decode(s):
    fa.flexattn_paged_decode(s["Q"], s["Kp"], s["Vp"], s["table"], s["ctx"], s["score"], s["mask"], s["params"],
                             s["scale"], s["O"], s["LSE"], s["ws"])
    return {"O": s["O"], "LSE": s["LSE"]}


def run(state):
    return {"train": _run_train, "prefill": _run_prefill, "decode": _run_decode}[state["case"]["kind"]](state)


# ---- what a pass cannot do without ----------------------------------------------------------------
def _pairs(case):
    """Unmasked (query, key) pairs of one head of one sequence; packed documents: of one drawn packing."""
    S, mask = case["S"], case["mask"]
    if mask == "none":
        return float(S * S)
    if mask == "neighborhood":
        return float(S * case["kernel"] ** 2)
    if mask == "documents":
        lengths = _document_lengths(random.Random(7), S, case["doc_min"], case["doc_max"])
        return float(sum(n * (n + 1) // 2 for n in lengths))
    q = torch.arange(S, dtype=torch.int64)
    first = torch.clamp(q - case["window"], min=0) if "window" in mask else torch.zeros_like(q)
    prefix = min(case["prefix_len"], S) if "prefix" in mask else 0
    keys = torch.where(first <= prefix, torch.clamp(q + 1, min=prefix), prefix + q + 1 - first)
    return float(keys.sum())


def work(case):
    if case["kind"] == "train":
        rows_q, rows_kv = case["B"] * case["Hq"] * case["S"], case["B"] * case["Hkv"] * case["S"]
        pairs = case["B"] * case["Hq"] * _pairs(case)
        row = 2 * case["D"]
        # read Q, K, V; write O, LSE; with gradients also read dO; write dQ, dK, dV
        nbytes = row * (2 * rows_q + 2 * rows_kv) + 4 * rows_q
        flops = 4 * case["D"] * pairs
        if case["backward"] != "none":
            nbytes += row * (2 * rows_q + 2 * rows_kv)
            flops += 10 * case["D"] * pairs
        return {"bytes": nbytes, "flops": flops}
    heads = case["Hq"], case["Hkv"]
    row = 2 * case["D"]
    if case["kind"] == "prefill":
        cached = 0.5 * (case["cached_min"] + case["cached_max"])
        n = case["chunk"]
        pairs = case["nseq"] * heads[0] * n * (cached + 0.5 * (n + 1))
        return {"bytes": case["nseq"] * (row * (2 * heads[0] * n + 2 * heads[1] * (cached + n)) + 4 * heads[0] * n),
                "flops": 4 * case["D"] * pairs}
    ctx = 0.5 * (case["ctx_min"] + case["ctx_max"])
    if case["window"] >= 0:
        ctx = min(ctx, case["window"] + 1)
    return {"bytes": case["nseq"] * (row * (2 * heads[0] + 2 * heads[1] * ctx) + 4 * heads[0]),
            "flops": 4 * case["D"] * case["nseq"] * heads[0] * ctx}


def tolerance(case):
    """bf16 operands and results, fp32 sums; the BlockMask's integers are the same.  Against the definition
    in 64 bits (B = 1, 2 to 4 heads, lengths of 1000 to 3000, every score_mod) the relative error of O and
    of every gradient is 2.1e-3 to 2.6e-3 (rounding a result to bf16 alone gives 1.7e-3); the largest
    difference over the root mean square is 7e-3 (decode), 3e-2 (forward) and 0.13 (gradients).  About four
    times each."""
    if case["kind"] == "decode":
        return {"rel": 8e-3, "max": 0.03}
    if case["kind"] == "prefill" or case["backward"] == "none":
        return {"rel": 9e-3, "max": 0.12}
    return {"rel": 1e-2, "max": 0.4}
