"""The work a user of the library has it do, as cases that can be timed and compared.

Four kinds of calls, all through the public entry points of `paper_2506_10848_amd.binding`:

  decode    `Model.decode` / `Model.decode_low_confidence`: a whole generation, the host's stage controller included
  step      `Model.step` / `Model.step_cached`: one denoising step of a caller that runs its own loop
  forward   `Model.forward`: bf16 logits of every position (scoring, or a sampler of the caller's own)
  select    `select`: the selector alone on logits that another program produced

Model shapes are the ones of `synth.CONFIGS` (tiny, medium, llada8b) with all their layers.

No trained weights exist here, so the weights are random with one thing planted that a trained model has: predictions
with a clear first choice, some positions nearly certain and the others far from it.  The embedding of a position
carries the id it is to predict (`_drafts` below) through the residual stream, the vocabulary projection recognises it
with a strength that depends on the id, and everything else (attention, feed-forward, all other ids) is random.  With
plain random weights every prediction would be a near tie that the last bit of a sum decides.
"""
import math

import numpy as np
import torch

from paper_2506_10848_amd import binding, synth

DEV = "cuda"
TAU_MIN, TAU_HIGH = 0.1, 0.9          # thresholds of the paper's runs
EMBED_STD = 4.0                       # the residual stream stays mostly the embedding, as in a trained model
# logit of the recognised id over the log-sum of the others: certain ids 0.98 to 0.998, uncertain ones 0.008 to 0.03;
# one id stands out, so that "the most confident position" is never a tie
CERTAIN, UNCERTAIN, TOP = (4.2, 6.2), (-4.8, -3.6), 9.0
TOP_ID = 1


def listed():
    return [
        # a whole generation by the smallest model: launch latency and the host loop are all there is
        dict(name="decode_tiny", kind="decode", model="tiny", batch=1, prompt=32, gen=64, uncertain=24,
             prompt_interval=0, response_interval=0, out_of_span=False, blocks=0, n_steps=0),
        # the service case of a small model: four sequences, prompt and response caches on as in the paper's Table 4
        dict(name="decode_medium_cached", kind="decode", model="medium", batch=4, prompt=128, gen=256, uncertain=45,
             prompt_interval=25, response_interval=5, out_of_span=True, blocks=0, n_steps=0),
        # the baseline sampler in four blocks, an odd prompt length
        dict(name="decode_medium_baseline", kind="decode", model="medium", batch=3, prompt=117, gen=132, uncertain=60,
             prompt_interval=0, response_interval=0, out_of_span=False, blocks=4, n_steps=32),
        # the benchmark's step: 8B model, one sequence, slow stage over the whole generated region
        dict(name="step_8b", kind="step", model="llada8b", batch=1, prompt=256, gen=256, span=0, skip=""),
        # a short odd sequence in the fast stage
        dict(name="step_8b_short", kind="step", model="llada8b", batch=1, prompt=75, gen=62, span=32, skip=""),
        # several sequences of odd length in one forward
        dict(name="step_8b_batch", kind="step", model="llada8b", batch=4, prompt=301, gen=256, span=0, skip=""),
        # long context and batch: the largest step
        dict(name="step_8b_long", kind="step", model="llada8b", batch=8, prompt=512, gen=1024, span=0, skip=""),
        # fast stage with prompt and out-of-span positions cached: only the span is recomputed (the weights are the work)
        dict(name="cached_8b_span", kind="step", model="llada8b", batch=1, prompt=256, gen=256, span=32, skip="prompt+rest"),
        # out-of-span caching alone: prompt and span are recomputed
        dict(name="cached_8b_prompt_span", kind="step", model="llada8b", batch=1, prompt=256, gen=256, span=32, skip="rest"),
        # logits of a whole sequence
        dict(name="forward_8b", kind="forward", model="llada8b", batch=1, prompt=384, gen=384),
        # the selector on a batch of long sequences
        dict(name="select_16x2048", kind="select", batch=16, length=2048, vocab=126464, masked=0.5, span=0),
        # and on one short sequence with a vocabulary whose rows are not aligned
        dict(name="select_odd_vocab", kind="select", batch=1, length=301, vocab=50257, masked=0.6, span=96),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "step", "step", "step", "cached", "cached", "forward", "select"])
    if kind == "decode":
        model = rng.choice(["tiny", "medium"])
        gen = 4 * rng.randint(6, 16) if model == "tiny" else 4 * rng.randint(16, 64)
        caches = model == "medium" and rng.random() < 0.5
        baseline = not caches and rng.random() < 0.4
        return dict(kind=kind, model=model, batch=rng.randint(1, 4), prompt=_log_int(rng, 9, 160), gen=gen,
                    uncertain=min(rng.randint(8, 48), gen // 2), prompt_interval=rng.randint(8, 40) if caches else 0,
                    response_interval=rng.randint(2, 8) if caches else 0, out_of_span=caches,
                    blocks=4 if baseline else 0, n_steps=4 * rng.randint(4, 10) if baseline else 0)
    if kind == "step":
        batch = rng.choice([1, 1, 1, 2, 3, 4, 6, 8])
        length = min(_log_int(rng, 64, 1536), 12288 // batch)
        gen = max(20, int(length * rng.uniform(0.3, 0.7)))
        return dict(kind=kind, model="llada8b", batch=batch, prompt=length - gen, gen=gen,
                    span=rng.choice([0, 0, min(gen, rng.randint(12, 96))]), skip="")
    if kind == "cached":
        gen = rng.randint(64, 512)
        return dict(kind="step", model="llada8b", batch=rng.choice([1, 1, 2]), prompt=rng.randint(40, 500), gen=gen,
                    span=rng.randint(12, 64), skip=rng.choice(["rest", "prompt+rest"]))
    if kind == "forward":
        length = _log_int(rng, 48, 1024)
        return dict(kind=kind, model="llada8b", batch=rng.choice([1, 1, 2]), prompt=length // 2, gen=length - length // 2)
    vocab = rng.choice([2048, 32000, 50257, 126464])
    batch = rng.choice([1, 2, 5, 16])
    length = min(_log_int(rng, 96, 2048), 16 * 2048 * 126464 // (batch * vocab))
    return dict(kind=kind, batch=batch, length=length, vocab=vocab, masked=round(rng.uniform(0.3, 0.9), 2),
                span=rng.choice([0, length // 3]))


# ---- inputs -------------------------------------------------------------------------------------------------------

def _normal(gen, shape, std):
    return torch.empty(shape, dtype=torch.bfloat16, device=DEV).normal_(0.0, std, generator=gen)


def _model_weights(cfg, gen):
    """Random weights (std 0.02, the projections that write the residual stream scaled down with depth) with the
    recognition of a position's own id planted in the vocabulary projection."""
    d, f, V, nl = cfg["d_model"], cfg["d_ffn"], cfg["vocab"], cfg["n_layers"]
    out_std = 0.02 / math.sqrt(2 * nl)
    gains = lambda: _normal(gen, (d,), 0.1).add_(1.0)
    w = dict(embed=_normal(gen, (V, d), EMBED_STD), lm_head=_normal(gen, (V, d), 0.02), final_norm=torch.ones(d, dtype=torch.bfloat16, device=DEV),
             attn_norm=[gains() for _ in range(nl)], ffn_norm=[gains() for _ in range(nl)],
             wqkv=[_normal(gen, (3 * d, d), 0.02) for _ in range(nl)], wo=[_normal(gen, (d, d), out_std) for _ in range(nl)],
             w_gate_up=[_normal(gen, (2 * f, d), 0.02) for _ in range(nl)], w_down=[_normal(gen, (d, f), out_std) for _ in range(nl)])
    # ids divisible by 4 are the uncertain ones (see _drafts)
    u = torch.rand((V,), device=DEV, generator=gen)
    sure = torch.arange(V, device=DEV) % 4 != 0
    over = torch.where(sure, CERTAIN[0] + u * (CERTAIN[1] - CERTAIN[0]), UNCERTAIN[0] + u * (UNCERTAIN[1] - UNCERTAIN[0]))
    over[TOP_ID] = TOP
    target = math.log(V) + 0.5 * 0.0004 * d + over
    for r in range(0, V, 16384):     # (in pieces: the fp32 products stay small)
        own, head = w["embed"][r:r + 16384].float() / EMBED_STD, w["lm_head"][r:r + 16384]
        head += (own * ((target[r:r + 16384] - (own * head).sum(1)) / d)[:, None]).to(torch.bfloat16)
    return w


def _drafts(cfg, batch, n, uncertain, rng):
    """Ids of n masked positions: `uncertain` of them the model is to be unsure of, one that stands out in the first
    quarter, and a certain one at the end (so that the first candidate span of a decode covers everything)."""
    ids = np.empty((batch, n), np.int32)
    quarter = cfg["vocab"] // 4 - 64
    for b in range(batch):
        ids[b] = 4 * rng.integers(1, quarter, n) + rng.integers(1, 4, n)
        places = rng.permutation(n - 1)
        top = int(places[places < max(2, n // 4)][0])
        ids[b, top] = TOP_ID
        at = places[places != top][:uncertain]
        ids[b, at] = 4 * rng.integers(1, quarter, len(at))
    ids[ids == cfg["mask_id"]] += 1
    return ids


def _model_state(case, seed):
    cfg = synth.CONFIGS[case["model"]]
    mc = synth.model_config(cfg)
    B, P, G = case["batch"], case["prompt"], case["gen"]
    L = P + G
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    rng = np.random.default_rng(seed)
    weights = _model_weights(cfg, gen)
    tokens = np.empty((B, L), np.int32)
    tokens[:, :P] = rng.integers(2, mc["mask_id"] - 2, (B, P))
    tokens[:, P:] = _drafts(cfg, B, G, min(case.get("uncertain", G * 2 // 5), G - 4), rng)
    mask = np.zeros((B, L), np.uint8)
    mask[:, P:] = 1
    s = dict(case=case, B=B, P=P, G=G, L=L, mc=mc, weights=weights, tokens0=torch.from_numpy(tokens).to(DEV),
             mask0=torch.from_numpy(mask).to(DEV), model=binding.Model(mc, weights, B, L))
    for k in ("tokens", "mask"):
        s[k] = s[k + "0"].clone()
    return s


def prepare(case, seed):
    if case["kind"] == "select":
        return _select_state(case, seed)
    s = _model_state(case, seed)
    B, P, G, L = s["B"], s["P"], s["G"], s["L"]
    if case["kind"] == "decode":
        s["params"] = binding.DecodeParams(10 ** 6, 8, 2, 1, 1, 1, 1.0, TAU_MIN, TAU_HIGH, int(case["out_of_span"]),
                                           case["prompt_interval"], case["response_interval"])
    elif case["kind"] == "step":
        s["prev0"] = torch.where(s["mask0"].bool(), s["tokens0"], torch.full_like(s["tokens0"], -1))   # the step before agreed
        s["prev"] = s["prev0"].clone()
        s["out"] = binding.CommitList(B, L)
        end = P + (case["span"] or G) - 1
        stage = binding.STAGE_FAST if case["span"] else binding.STAGE_SLOW
        s["end"] = end
        s["sps"] = [binding.stage_params(stage, P, end, 1, TAU_MIN, TAU_HIGH, 1, P, L) for _ in range(B)]
        if case["skip"]:
            skip = np.zeros((B, L), np.uint8)
            skip[:, end + 1:] = 1
            if case["skip"].startswith("prompt"):
                skip[:, :P] = 1
            s["skip"] = skip
            # the complete first step of the fast stage fills the key/value cache; the steps after it are the case
            s["model"].step_cached(s["tokens"], s["mask"], s["prev"], s["sps"], [binding.CACHE_REFRESH] * B, None, s["out"])
    return s


def _select_state(case, seed):
    """Logits N(0, 1) with a peak at one id per position: one half of them 2 to 8 (nothing decided), the other half 13.8
    to 18 (certain); previous predictions that agree with the current ones on 70 % of the positions."""
    B, L, V = case["batch"], case["length"], case["vocab"]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    logits = torch.empty((B, L, V), dtype=torch.bfloat16, device=DEV)
    for b in range(B):
        logits[b].normal_(0.0, 1.0, generator=gen)
    rand = lambda: torch.rand((B, L), device=DEV, generator=gen)
    mask_id = V - 1 - V // 1000
    planted = (rand() * (mask_id - 1)).to(torch.int64)
    peak = torch.where(rand() < 0.5, 2 + 6 * rand(), 13.8 + 4.2 * rand())
    at = logits.gather(2, planted[..., None]).float() + peak[..., None]
    logits.scatter_(2, planted[..., None], at.to(torch.bfloat16))
    mask0 = (rand() < case["masked"]).to(torch.uint8)
    prev0 = torch.where(rand() < 0.7, planted, (planted + 1) % mask_id).to(torch.int32)
    tokens0 = torch.where(mask0.bool(), torch.full_like(prev0, mask_id), planted.to(torch.int32))
    stage, end = (binding.STAGE_FAST, case["span"] - 1) if case["span"] else (binding.STAGE_SLOW, L - 1)
    return dict(case=case, B=B, L=L, logits=logits, mask_id=mask_id, mask0=mask0, prev0=prev0, tokens0=tokens0, mask=mask0.clone(),
                prev=prev0.clone(), tokens=tokens0.clone(), pred=torch.zeros_like(prev0), out=binding.CommitList(B, L),
                conf=torch.zeros((B, L), dtype=torch.float32, device=DEV),
                sps=[binding.stage_params(stage, 0, end, 1, TAU_MIN, TAU_HIGH, 1, 0, L) for _ in range(B)])


# ---- one pass -----------------------------------------------------------------------------------------------------

def _commits(out):
    return [out.n_commit, out.pos, out.tok, out.conf, out.e_cand, out.first_masked, out.n_masked_after]


def _held(view, model):
    """A view of the handle's workspace that keeps the handle alive."""
    view.owner = model
    return view


def run(s):
    kind = s["case"]["kind"]
    if kind == "forward":
        return _held(s["model"].forward(s["tokens0"]), s["model"])
    s["tokens"].copy_(s["tokens0"])       # the next request: its tokens and mask go to where the program keeps them
    s["mask"].copy_(s["mask0"])
    if kind == "decode":
        if s["case"]["blocks"]:
            steps, _ = s["model"].decode_low_confidence(s["tokens"], s["mask"], s["P"], s["case"]["n_steps"], s["G"] // s["case"]["blocks"])
        else:
            steps, _ = s["model"].decode(s["tokens"], s["mask"], s["P"], s["params"])
        return s["tokens"], s["mask"], steps
    s["prev"].copy_(s["prev0"])
    if kind == "select":
        binding.select(s["logits"], s["tokens"], s["mask"], s["prev"], s["sps"], s["mask_id"], s["pred"], s["conf"], s["out"])
        return s["tokens"], s["mask"], s["prev"], s["pred"], s["conf"], _commits(s["out"])
    if s["case"]["skip"]:
        s["model"].step_cached(s["tokens"], s["mask"], s["prev"], s["sps"], [binding.CACHE_REUSE] * s["B"], s["skip"], s["out"])
    else:
        s["model"].step(s["tokens"], s["mask"], s["prev"], s["sps"], s["out"])
    # every position of the window was masked, so all of its predictions and confidences are defined
    pred, conf = (_held(t.view(s["B"], s["L"])[:, s["P"]:s["end"] + 1], s["model"]) for t in s["model"].debug_rows(s["B"] * s["L"]))
    return s["tokens"], s["mask"], s["prev"], pred, conf, _commits(s["out"])


# ---- what a pass cannot do without --------------------------------------------------------------------------------

def _pass_work(cfg, rows, rated, pairs, kv_rows=0):
    """One forward over `rows` positions: every weight read once, flops of the projections, of attention over `pairs`
    (query, key) pairs and of the vocabulary projection of `rated` positions; kv_rows: cached positions read per layer."""
    d, f, V, nl = cfg["d_model"], cfg["d_ffn"], cfg["vocab"], cfg["n_layers"]
    weights = nl * (4 * d * d + 3 * d * f) + V * d
    return dict(bytes=2.0 * weights + 2.0 * rows * d + nl * 4.0 * kv_rows * d,
                flops=2.0 * rows * nl * (4 * d * d + 3 * d * f) + 2.0 * rated * d * V + 4.0 * nl * pairs * d)


def work(case):
    if case["kind"] == "select":
        rated = case["batch"] * (case["span"] or case["length"]) * case["masked"]
        return dict(bytes=2.0 * rated * case["vocab"] + 9.0 * case["batch"] * case["length"], flops=4.0 * rated * case["vocab"])
    cfg = synth.CONFIGS[case["model"]]
    B, P, G = case["batch"], case["prompt"], case["gen"]
    L = P + G
    if case["kind"] == "forward":
        w = _pass_work(cfg, B * L, B * L, B * L * L)
        w["bytes"] += 2.0 * B * L * cfg["vocab"]
        return w
    if case["kind"] == "step":
        rated = B * (case["span"] or G)
        rows = B * L if not case["skip"] else rated + (0 if case["skip"].startswith("prompt") else B * P)
        return _pass_work(cfg, rows, rated, rows * L, B * L - rows if case["skip"] else 0)
    # a decode: two slow steps, one fast step that commits what is certain, then the uncertain positions one by one
    steps = case["n_steps"] or case["uncertain"] + 3
    rows, rated = B * L, B * G / (2.0 * (case["blocks"] or 1))
    if case["response_interval"]:        # between two refreshes of the response only the rated positions are recomputed
        rows = B * G / case["response_interval"] + rated * (1 - 1.0 / case["response_interval"])
    w = _pass_work(cfg, rows, rated, rows * L, B * L - rows)
    return {k: v * steps for k, v in w.items()}


def tolerance(case):
    if case["kind"] == "select":       # one fp32 sum over a vocabulary in another order
        return {"rel": 1e-5, "max": 1e-4}
    if case["kind"] == "decode":       # ids and steps of clear decisions
        return "exact"
    # about four times what the same forward differs by with its RMSNorm in another place and its sums split otherwise
    # (confidences 1.5e-3, largest 2e-2; logits 3.4e-3, 1.8e-2); bf16 activations over 32 layers
    return {"rel": 0.014, "max": 0.08} if case["kind"] == "forward" else {"rel": 0.006, "max": 0.08, "differ": 0.002}
