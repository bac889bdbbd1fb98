"""The work a user of this library has it do, as cases that can be timed: block-decode steps, first blocks of new prompts,
self-speculative steps and whole short generations, from one sequence of a small model to full batches of large ones.

A case names the shape of a decoder (the workloads of paper_2509_24007_amd/inputs.py), how many of its layers are present, and what is
done with it:
  step      one block-decode step of sequences that are under way: every sequence carries 1 to min(D, 3) accepted tokens of the
            step before (a trained model accepts about two), so the step runs batch * (D + 2) rows on average
  first     new prompts to their first predicted block: prefill, then one step
  selfspec  a step and the verification pass over its tokens
  generate  prefill and `steps` steps, each committing what it accepted
The wide shapes are cut in depth: the launches of a layer do not depend on how many follow, and ten preparations of a case
have to stay affordable.

Weights are drawn so that the values inside the decoder are those of a trained one: unit-scale activations in every layer (fan-in
scaling, residual projections scaled down with the depth, scores wide enough that a query rests on some tens of keys) and an
LM head on which the leading token stands out.  The head is the embedding table under a cyclic shift of the vocabulary, mixed
with noise: about half of the tokens are predicted with near certainty and half with a probability around one half.
Predictions on a random head would hang on ties that any rounding decides.
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2509_24007_amd import inputs as syn
from paper_2509_24007_amd import sdlm

SHAPES = {"tiny": "C1", "1.5B": "C2", "3B": "C3", "7B": "C4", "32B": "C5"}
DEPTHS = {"tiny": 2, "1.5B": 28, "3B": 36, "7B": 8, "32B": 4}      # layers of a drawn case; the whole model for the narrow ones


def _case(do, shape, layers, batch, lo, hi, D, *, tau=0.9, paged=False, conf_fn=0, static=False, steps=1, name=None):
    c = {"do": do, "shape": shape, "layers": layers, "batch": batch, "prompt_lo": lo, "prompt_hi": hi, "D": D, "tau": tau, "paged": paged,
         "conf_fn": conf_fn, "static": static, "steps": steps}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the tiny fp32 workload whole: the debug mode, and the cost of a call when there is next to nothing to compute
        _case("generate", "tiny", 2, 1, 64, 64, 4, tau=0.5, steps=32, name="tiny fp32 generate"),
        # one user of a small model: latency, launches, weight streaming with a handful of rows
        _case("step", "1.5B", 28, 1, 512, 512, 4, name="1.5B step b1"),
        # the same user's wait for the first block after a prompt of odd length
        _case("first", "1.5B", 28, 1, 509, 509, 4, name="1.5B first block b1"),
        # a small server's batch with larger blocks, contiguous cache
        _case("step", "3B", 36, 16, 1024, 2048, 8, name="3B step b16"),
        # the same batch decoding self-speculatively
        _case("selfspec", "3B", 36, 16, 1024, 2048, 8, name="3B selfspec b16"),
        # next-token decoding (block size 1) of an odd batch, for a caller that cannot lend scratch memory
        _case("step", "3B", 36, 33, 256, 768, 1, static=True, name="3B next-token b33 static"),
        # a few users of a 7B model at its whole depth: an odd batch, an odd block size, very different lengths, entropy confidence
        _case("step", "7B", 28, 7, 100, 3000, 5, paged=True, conf_fn=1, name="7B step b7 odd"),
        # the throughput workload whole: a full batch over a paged cache
        _case("step", "7B", 28, 64, 2048, 4096, 4, paged=True, name="7B step b64"),
        # several long prompts to their first block: matrix products over thousands of rows
        _case("first", "7B", 8, 6, 2048, 4096, 4, paged=True, name="7B first block b6"),
        # one user of a large model with a long context
        _case("step", "32B", 16, 1, 4096, 8192, 4, paged=True, name="32B step b1"),
        # a batch of long contexts on a large model: the cache alone is most of the traffic
        _case("step", "32B", 4, 32, 4096, 8192, 4, paged=True, name="32B step b32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    cap = max(_cost(c) for c in listed())
    while True:
        shape = rng.choice(["1.5B", "3B", "7B", "32B", "1.5B", "3B", "7B", "32B", "tiny"])
        do = "generate" if shape == "tiny" else rng.choice(["step"] * 6 + ["first"] * 2 + ["selfspec"])
        hi = _log_int(rng, 33, 8192 if shape != "tiny" else 256)
        lo = max(1, _log_int(rng, max(1, hi // 16), hi))
        batch = _log_int(rng, 1, 64) if shape != "tiny" else rng.choice([1, 1, 2, 3])
        D = rng.choice([1, 2, 3, 4, 4, 4, 4, 5, 6, 7, 8, 8, 11, 16])
        if do == "selfspec":
            D = min(max(D, 2), 8)
        if do == "first":
            batch = min(batch, max(1, 24000 // hi))
        static = do == "step" and batch * D <= 256 and rng.random() < 0.15
        c = _case(do, shape, DEPTHS[shape], batch, lo, hi, D, tau=rng.choice([0.5, 0.8, 0.9, 0.98]), paged=rng.random() < 0.6,
                  conf_fn=int(rng.random() < 0.25), static=static, steps=_log_int(rng, 4, 48) if do == "generate" else 1)
        # what the preparation costs is bounded too: prompt tokens times weights
        if batch * hi * _layer_elems(_model(c)) * c["layers"] > 6e14:
            continue
        if _cost(c) <= cap:
            return c


# ---------------------------------------------------------------------------------------------------------------- model and inputs

def _model(case):
    m = syn.workloads()[SHAPES[case["shape"]]].model
    return dataclasses.replace(m, n_layers=case["layers"], logit_scale=1.0)


def _load_weights(ctx, m, gen):
    dt, dev, V, h = m.torch_dtype, "cuda", m.vocab, m.hidden

    def normal(shape, std):
        return torch.empty(shape, dtype=dt, device=dev).normal_(0.0, std, generator=gen)

    embed = normal((V, h), 1.0)
    # logit of token t + 1 for input t is about lead * sqrt(h): level with all other tokens together, or well above them
    level = min(0.6, 1.1 * (math.log(V) + 0.5) / math.sqrt(h))
    strong = torch.rand(V, generator=gen, device=dev) < 0.5
    strong[m.mask_token_id] = True
    lead = torch.where(strong, min(2.0 * level, 0.98), level).roll(1).unsqueeze(1)
    head = torch.empty(V, h, dtype=dt, device=dev)
    for lo in range(0, V, 1 << 15):
        hi = min(V, lo + (1 << 15))
        src = torch.arange(lo - 1, hi - 1, device=dev) % V
        noise = torch.empty(hi - lo, h, device=dev).normal_(0.0, 1.0, generator=gen)
        a = lead[lo:hi]
        head[lo:hi] = ((a * embed[src].float() + torch.sqrt(1.0 - a * a) * noise) / math.sqrt(h)).to(dt)
    ctx.init_weights({"embed": embed, "lm_head": head, "final_norm": torch.ones(h, dtype=dt, device=dev)}, None)
    del embed, head
    for l in range(m.n_layers):
        L = {}
        for name, shape in syn.layer_shapes(m).items():
            if name in ("attn_norm", "ffn_norm"):
                L[name] = torch.ones(shape, dtype=dt, device=dev)
            elif name in ("bq", "bk", "bv"):
                L[name] = normal(shape, 0.1) if m.has_qkv_bias else None
            else:
                gain = 1.5 if name in ("wq", "wk") else 1.0 / math.sqrt(2 * m.n_layers) if name in ("wo", "w_down") else 1.0
                L[name] = normal(shape, gain / math.sqrt(shape[1]))
        ctx.init_weights(None, {l: L})


def prepare(case, seed):
    m, B, D, V = _model(case), case["batch"], case["D"], syn.workloads()[SHAPES[case["shape"]]].model.vocab
    rng = np.random.default_rng([seed, 1])
    gen = torch.Generator(device="cuda").manual_seed(seed)
    lens = rng.integers(case["prompt_lo"], case["prompt_hi"] + 1, B)
    prompts = [rng.integers(0, V, int(n), dtype=np.int32) for n in lens]
    max_len = int(max(lens)) + (case["steps"] + 2) * D
    n_pages = sum((int(n) + (case["steps"] + 2) * D + 15) // 16 for n in lens) if case["paged"] else 0
    ctx = sdlm.Context(sdlm.model_cfg(m), max_batch=B, max_seq_len=max_len, block_D=D, tau=case["tau"], paged=case["paged"], n_pages=n_pages,
                       conf_fn=case["conf_fn"])
    _load_weights(ctx, m, gen)
    n = case["steps"]
    s = {"case": case, "ctx": ctx, "prompts": prompts,
         "ids": torch.zeros(n, B, D, dtype=torch.int32, device="cuda"), "count": torch.zeros(n, B, dtype=torch.int32, device="cuda"),
         "conf": torch.zeros(n, B, D, device="cuda"), "logits": torch.zeros(n, B, D, V, device="cuda")}
    if case["do"] == "selfspec":
        s["tilde"] = torch.zeros(B, D, dtype=torch.int32, device="cuda")
        s["verified"] = torch.zeros(B, dtype=torch.int32, device="cuda")
        s["verify_logits"] = torch.zeros(B, D - 1, V, device="cuda")
    if case["do"] in ("step", "selfspec"):
        ctx.prefill(prompts)
        ctx.decode_step(s["ids"][0], s["count"][0])
        ctx.kv_commit(torch.from_numpy(rng.integers(0, V, (B, D), dtype=np.int32)).cuda(),
                      torch.from_numpy(rng.integers(1, min(D, 3) + 1, B, dtype=np.int32)).cuda())
    return s


def run(state):
    ctx, case = state["ctx"], state["case"]
    if case["do"] in ("first", "generate"):
        ctx.prefill(state["prompts"])
    for t in range(case["steps"]):
        ctx.decode_step(state["ids"][t], state["count"][t], state["conf"][t], state["logits"][t], static_scratch=case["static"])
        if case["do"] == "generate":
            ctx.kv_commit()
    out = [state["ids"], state["count"], state["conf"], state["logits"]]
    if case["do"] == "selfspec":
        ctx.verify_step(0, state["tilde"], state["verified"], state["verify_logits"])
        out += [state["tilde"], state["verified"], state["verify_logits"]]
    return out


# ---------------------------------------------------------------------------------------------------------------- work and tolerance

def _layer_elems(m):
    nq, nk = m.n_q_heads * m.head_dim, m.n_kv_heads * m.head_dim
    return m.hidden * (nq + 2 * nk) + nq * m.hidden + 3 * m.hidden * m.ffn


def work(case):
    """Every weight once per pass over the model, every cached key and value once, new ones written once, logits written once."""
    m, B, D, L = _model(case), case["batch"], case["D"], case["layers"]
    e = 4 if m.dtype == "fp32" else 2
    qd, kd, V, h = m.n_q_heads * m.head_dim, m.n_kv_heads * m.head_dim, m.vocab, m.hidden
    mean = (case["prompt_lo"] + case["prompt_hi"]) / 2.0
    pending = (1 + min(D, 3)) / 2.0
    bytes_ = flops = 0.0

    def layers(rows, keys):      # `keys`: keys that a row sees, averaged over the rows
        return 2.0 * rows * L * _layer_elems(m) + 4.0 * rows * keys * L * qd

    def head(rows):
        return 2.0 * rows * V * h, V * h * e + rows * V * 4.0

    if case["do"] in ("first", "generate"):
        tokens = B * mean
        flops += layers(tokens, mean / 2)
        bytes_ += L * _layer_elems(m) * e + tokens * (h * e + 2 * kd * L * e)
        pending = 0.0
    for t in range(case["steps"]):
        rows = B * (D + (1.0 if t else pending))
        f, b = head(B * D)
        flops += layers(rows, mean) + f
        bytes_ += L * _layer_elems(m) * e + b + B * mean * 2 * kd * L * e + rows * h * e + B * 2 * kd * L * e
    if case["do"] == "selfspec":
        rows = B * ((D - 2) + (D - 1) * D)
        f, b = head(B * (D - 1))
        flops += layers(rows, mean) + f
        bytes_ += L * _layer_elems(m) * e + b + B * mean * 2 * kd * L * e + rows * h * e
    return {"bytes": bytes_, "flops": flops}


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 300.0)


def tolerance(case):
    """Measured on the listed cases between two correct paths of the library: a sequence in its batch and alone, scratch in the
    workspace and static, prompts in passes of 64 and of 4096 rows.  bf16: logits differ by 2.1e-3 to 3.1e-3 in the 2-norm and by at most 1.5e-2
    at one value; four times that.  fp32: the size of another order of the sums."""
    if case["shape"] == "tiny":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 0.012, "max": 0.06}
