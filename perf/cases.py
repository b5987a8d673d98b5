"""The work that a user of this library has it do, as cases that can be timed and compared.

A case names a kind of call, one of the repository's model shapes (at the full width, with as many
layers as keep a pass short), and how many samples of which lengths it runs over:

  stage     the whole stage: rlhf_submit, rlhf_run_stage (plan chosen by the library), rlhf_get_results;
            Actor generation fused with the Reference, Critic and Reward scoring forwards
  generate  the generation stage alone (one role): prefill of every prompt, then decode steps
  prefill   admission of a batch of prompts: the step that yields every sample's first token
  score     rlhf_score of a finished batch by Reference, Critic and Reward, and its results
  gae       rlhf_compute_gae over a finished stage

Weights are N(0, 0.02^2), prompts uniform over the vocabulary.  Response tokens are imposed (recorded
rollouts replayed through forced_tokens), because one greedy choice decided the other way by rounding
would change everything generated after it; the pick kernels run all the same.  In `generate` the last
token of every sample is free, so that its greedy choice is part of the outputs, where outputs are long
enough for a near-tie among those last tokens to stay within the share that may differ.

Lengths are the quantiles of the shape's length law (prompts: even steps over its prompt range), in an
order drawn from the seed, so that every seed asks for the same amount of work.
"""
import math

import numpy as np
import torch

import paper_2409_13221_amd as R

PAGE = 16
EOS = 2
MAX_BATCH_TOKENS = 8192          # rows of one prefill / scoring pass, as the benchmark sets it
SCORE_ROLES = 0b1110             # Reference, Critic, Reward

# the repository's five model shapes: widths, prompt range, output-length law
SHAPES = {
    "tiny": dict(d=256, hq=4, hkv=4, hd=64, ffn=688, vocab=4096, dtype="fp32", prompt=(32, 32),
                 law="lognormal", params=(3.0, 0.8)),
    "gpt2s": dict(d=768, hq=12, hkv=12, hd=64, ffn=2048, vocab=32000, dtype="bf16", prompt=(256, 256),
                  law="lognormal", params=(4.8, 1.0)),
    "7b": dict(d=4096, hq=32, hkv=32, hd=128, ffn=11008, vocab=32000, dtype="bf16", prompt=(128, 512),
               law="pareto", params=(1.5, 64.0)),
    "13b": dict(d=5120, hq=40, hkv=40, hd=128, ffn=13824, vocab=32000, dtype="bf16", prompt=(512, 512),
                law="pareto", params=(1.2, 128.0)),
    "70b_slice": dict(d=8192, hq=64, hkv=8, hd=128, ffn=28672, vocab=32000, dtype="bf16", prompt=(1024, 1024),
                      law="lognormal", params=(6.0, 1.0)),
}


def _case(name, kind, model, layers, samples, new, law=False, prompt=None, half=True):
    lo, hi = prompt or SHAPES[model]["prompt"]
    c = {"kind": kind, "model": model, "layers": layers, "samples": samples, "prompt_lo": lo, "prompt_hi": hi,
         "new": new, "law": law, "half_copies": half and SHAPES[model]["dtype"] == "bf16"}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest configuration, float32, every step a chain of small launches: what a first user runs
        _case("tiny_stage", "stage", "tiny", 2, 8, 64, law=True),
        # a small bf16 model at full depth; decode steps bound by their launches
        _case("gpt2s_stage", "stage", "gpt2s", 12, 64, 192, law=True),
        # the benchmark's mixture at its width: long-tailed outputs, scoring overlapped with decoding
        _case("7b_stage", "stage", "7b", 4, 64, 512, law=True),
        # the end of the long tail: one sample left, the latency of a decode step, full depth
        _case("7b_generate_1", "generate", "7b", 32, 1, 112),
        # a handful of samples, where a step's time is still its weights
        _case("7b_generate_13", "generate", "7b", 16, 13, 64),
        # the middle of a batch
        _case("7b_generate_64", "generate", "7b", 8, 64, 96),
        # the whole batch active, as at the start of every stage: weights, KV and matrix work all count
        _case("7b_generate_256", "generate", "7b", 4, 256, 64),
        # grouped KV heads, wide layers, contexts past a thousand tokens
        _case("70b_generate_32", "generate", "70b_slice", 2, 32, 96),
        # admission of a full batch pass; bf16 weights as a caller binds them, no half copies
        _case("7b_prefill", "prefill", "7b", 8, 25, 1, half=False),
        # one scoring batch of the benchmark's size by the three scoring models
        _case("7b_score", "score", "7b", 8, 17, 512, law=True),
        # long sequences, where packed causal attention carries weight beside the projections
        _case("13b_score", "score", "13b", 3, 5, 1024, law=True, prompt=(512, 2047)),
        # advantages and returns of a whole benchmark batch, long tail included
        _case("gae_256", "gae", "tiny", 1, 256, 2048, law=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    limit = 0.6 * max(_seconds(c) for c in listed())
    while True:
        kind = rng.choice(("stage", "generate", "generate", "generate", "prefill", "score", "score", "gae"))
        model = rng.choice(tuple(SHAPES))
        if kind == "gae":
            c = _case(None, kind, "tiny", 1, _log_int(rng, 3, 384), _log_int(rng, 24, 2048), law=True)
        else:
            deepest = {"tiny": 2, "gpt2s": 12, "7b": 8, "13b": 4, "70b_slice": 2}[model]
            lo = _log_int(rng, 12, 768)
            c = _case(None, kind, model, rng.randint(1, deepest), _log_int(rng, 1, 256),
                      1 if kind == "prefill" else _log_int(rng, 9, 512), law=kind in ("stage", "score"),
                      prompt=(lo, lo + _log_int(rng, 1, 1024)), half=rng.random() < 0.7)
        if 2e-3 < _seconds(c) < limit and _prepare_seconds(c) < 1.0:
            return c


# ---------------------------------------------------------------------------------- lengths and work

_NORMAL = None


def _quantiles(case):
    """Output lengths of the case, ascending."""
    global _NORMAL
    n, cap, s = case["samples"], case["new"], SHAPES[_law_of(case)]
    if not case["law"]:
        return np.full(n, cap, np.int64)
    u = (np.arange(n) + 0.5) / n
    a, b = s["params"]
    if s["law"] == "pareto":
        raw = np.floor(b * (1.0 - u) ** (-1.0 / a))
    else:
        if _NORMAL is None:
            from statistics import NormalDist
            _NORMAL = NormalDist()
        raw = np.rint(np.exp(a + b * np.array([_NORMAL.inv_cdf(float(x)) for x in u])))
    return np.clip(raw, 1, cap).astype(np.int64)


def _law_of(case):
    return "7b" if case["kind"] == "gae" else case["model"]      # GAE: the benchmark's lengths over a small model


def _prompts(case):
    return np.rint(np.linspace(case["prompt_lo"], case["prompt_hi"], case["samples"])).astype(np.int64)


def _layer_params(s):
    return (s["hq"] + 2 * s["hkv"]) * s["hd"] * s["d"] + s["d"] * s["hq"] * s["hd"] + 3 * s["d"] * s["ffn"]


def _pass_flops(case, tokens, seq):
    """A causal forward over `tokens` rows in sequences of mean length `seq` (heads not included)."""
    s = SHAPES[case["model"]]
    return case["layers"] * tokens * (2.0 * _layer_params(s) + 4.0 * s["hq"] * s["hd"] * (seq + 1) / 2)


def work(case):
    s, L = SHAPES[case["model"]], case["layers"]
    es = 4 if s["dtype"] == "fp32" else 2
    P, G = _prompts(case), _quantiles(case)
    n, tp, tg = case["samples"], float(P.sum()), float(G.sum())
    if case["kind"] == "gae":        # three float results per token in, two out
        return {"bytes": 20.0 * tg + 4.0 * n, "flops": 8.0 * tg}
    weights = (L * _layer_params(s) + s["vocab"] * s["d"]) * es
    head = 2.0 * s["vocab"] * s["d"]
    kv_tok = 2.0 * L * s["hkv"] * s["hd"] * es
    nbytes = flops = 0.0
    if case["kind"] != "score":
        passes = math.ceil(tp / MAX_BATCH_TOKENS)
        nbytes += passes * weights + tp * kv_tok + 4.0 * tp
        flops += _pass_flops(case, tp, float((P * P).sum()) / tp) + head * n
        steps = int(G.max()) - 1
        rows = tg - n                                       # decode inputs
        ctx = float(P.mean() * rows + ((G - 1) * G / 2.0).sum())   # cached tokens read, over all rows
        nbytes += steps * weights + ctx * kv_tok + rows * kv_tok + 8.0 * tg
        flops += rows * (2.0 * L * _layer_params(s) + head) + 4.0 * L * s["hq"] * s["hd"] * ctx
    if case["kind"] in ("stage", "score"):
        T = tp + tg
        seq = float(((P + G.mean()) ** 2).sum()) / T
        passes = math.ceil(T / MAX_BATCH_TOKENS)
        nbytes += passes * (3 * L * _layer_params(s) + s["vocab"] * s["d"]) * es + 3 * 4.0 * T + 8.0 * tg
        flops += 3 * _pass_flops(case, T, seq) + head * tg
    return {"bytes": nbytes, "flops": flops}


def _seconds(case):
    """A rough estimate of a pass, for choosing what to draw."""
    w, s = work(case), SHAPES[case["model"]]
    rate = 5e12 if s["dtype"] == "fp32" else 8e14
    steps = int(_quantiles(case).max())
    chain = steps * (10 * case["layers"] + 6) * 5e-6 if case["kind"] in ("stage", "generate") else 0.0
    return w["bytes"] / 4e12 + w["flops"] / rate + chain + 1e-3


def _prepare_seconds(case):
    s = SHAPES[case["model"]]
    steps = int(_quantiles(case).max()) if case["kind"] in ("score", "gae") else 0
    rows = float(_quantiles(case).sum())
    t = steps * ((10 * case["layers"] + 6) * 5e-6 + case["layers"] * _layer_params(s) * 2 / 4e12)
    return t + rows * case["layers"] * _layer_params(s) * 2 / 2e14


def tolerance(case):
    # Four times what the path differs by from itself with its sums in another order (other tilings and
    # K splits, decode against a re-scoring forward).  Float32 models and GAE: values 7e-7, at most 2e-6.
    if case["kind"] == "gae":
        return {"rel": 2e-6, "max": 2e-5}
    if SHAPES[case["model"]]["dtype"] == "fp32":
        return {"rel": 5e-6, "max": 2e-5, "differ": 0.01}
    # bf16 models run half activations: log-probs differ by 1e-4 to 2e-4 of their size, values and rewards,
    # small numbers on top of the same hidden states, by 1e-3 (single entries by 4e-3).  A near-tie among
    # the free last tokens may fall either way.
    return {"rel": 5e-3, "max": 2e-2, "differ": 0.01}


# ------------------------------------------------------------------------------------ state and pass

class _Stage:
    """A context with its borrowed weights and the batch it runs over."""

    def __init__(self, case, seed):
        self.case = case
        s, L, n = SHAPES[case["model"]], case["layers"], case["samples"]
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed)
        wdt = torch.float32 if s["dtype"] == "fp32" else torch.bfloat16
        d, f, qd, kvd = s["d"], s["ffn"], s["hq"] * s["hd"], s["hkv"] * s["hd"]

        def normal(*shape):
            return torch.empty(shape, device="cuda", dtype=wdt).normal_(0.0, 0.02, generator=gen)

        def gains(*shape):
            return 1.0 + 0.05 * torch.empty(shape, device="cuda").normal_(generator=gen)

        roles = range(4) if case["kind"] in ("stage", "score", "gae") else range(1)
        self.weights = [{"embed": normal(s["vocab"], d), "wqkv": normal(L, qd + 2 * kvd, d), "wo": normal(L, d, qd),
                         "w_gate_up": normal(L, 2 * f, d), "w_down": normal(L, d, f), "g_attn": gains(L, d),
                         "g_mlp": gains(L, d), "g_final": gains(d), "head": normal(s["vocab"] if r < 2 else 1, d)}
                        for r in roles]
        torch.cuda.synchronize()             # the library's streams do not wait for torch's

        rng = np.random.default_rng(seed)
        self.plen = rng.permutation(_prompts(case))
        self.out_len = rng.permutation(_quantiles(case)).astype(np.int32)
        self.prompt_offsets = np.concatenate([[0], np.cumsum(self.plen)]).astype(np.int64)
        self.prompt_tokens = rng.integers(3, s["vocab"], int(self.plen.sum())).astype(np.int32)
        self.resp_offsets = np.concatenate([[0], np.cumsum(self.out_len)]).astype(np.int64)
        self.responses = rng.integers(3, s["vocab"], int(self.out_len.sum())).astype(np.int32)
        self.total = int(self.out_len.sum())
        free_last = case["kind"] == "generate" and (case["new"] >= 100 or (case["new"] >= 32 and n * case["new"] >= 200))
        if free_last:
            self.responses[self.resp_offsets[1:] - 1] = -1
        # without an imposed length a sample ends at its cap, and its last token is the greedy one
        self.forced_len = None if free_last else self.out_len

        page_bytes = L * 2 * kvd * PAGE * (4 if s["dtype"] == "fp32" else 2)
        # every sample's whole length, and the page per running sample that optimistic admission keeps free
        pages = int(-(-(self.plen + self.out_len + 1) // PAGE).sum()) + n
        max_ctx = int((self.plen + self.out_len).max()) + 1
        mc = R.rlhf_model_cfg(L, d, s["hq"], s["hkv"], s["hd"], f, s["vocab"],
                              R.RLHF_FP32 if s["dtype"] == "fp32" else R.RLHF_BF16, 1e-5, 10000.0)
        ec = R.rlhf_engine_cfg(PAGE, pages * page_bytes, n, max_ctx, n, max(MAX_BATCH_TOKENS, max_ctx), EOS, 0, 0, 1,
                               None, None, int(case["half_copies"]))
        self.ctx = R.rlhf_create(mc, ec)
        for role, w in enumerate(self.weights):
            R.rlhf_load_weights(self.ctx, role, w)

    def submit(self):
        R.rlhf_submit(self.ctx, self.prompt_tokens, self.prompt_offsets, self.out_len, self.forced_len, self.responses,
                      self.resp_offsets)

    def generate(self):
        R.rlhf_run_stage(self.ctx, False, 0, 1 << 30, 0)

    def __del__(self):
        if getattr(self, "ctx", None) is not None:
            R.rlhf_destroy(self.ctx)


def prepare(case, seed):
    st = _Stage(case, seed)
    if case["kind"] in ("score", "gae"):     # these start from a finished stage
        st.submit()
        if case["kind"] == "score":
            st.generate()
        else:
            R.rlhf_run_stage(st.ctx, "auto", st.case["samples"] + 1, MAX_BATCH_TOKENS, SCORE_ROLES)
    return st


def run(st):
    kind, n = st.case["kind"], st.case["samples"]
    if kind == "gae":
        adv, ret = R.rlhf_compute_gae(st.ctx, 0.99, 0.95, 0.05, st.total)
        return {"advantages": adv, "returns": ret}
    if kind == "score":
        R.rlhf_score(st.ctx, range(n), SCORE_ROLES)
    else:
        st.submit()
        if kind == "stage":
            R.rlhf_run_stage(st.ctx, "auto", n + 1, MAX_BATCH_TOKENS, SCORE_ROLES)
        elif kind == "generate":
            st.generate()
        else:
            R.rlhf_generate_step(st.ctx)
    res = R.rlhf_get_results(st.ctx, n, st.total)
    keys = ["lp_ref", "values", "reward"] if kind in ("stage", "score") else []
    if kind != "score":
        keys += ["tokens", "lp_actor"]
    return {k: res[k] for k in keys}
