"""GPU parity: the HIP library against the CPU oracle, element by element, through the C ABI."""
import json
import os

import numpy as np
import pytest
import torch

from gpu_common import both_models, gpu_context, lockstep
from helpers import make_model, small_cfg
from oracle import oracle as orc
from paper_2509_24007_amd import inputs as syn

pytestmark = pytest.mark.gpu
GOLD = os.path.join(os.path.dirname(__file__), "golden")


def gpu_cfg(**kw):
    base = dict(hidden=64, n_q_heads=4, n_kv_heads=2, head_dim=32, ffn=112, vocab=300)
    base.update(kw)
    return small_cfg(**base)


def test_c1_tiny_fp32_free_running():
    """The tiny fp32 workload: 32 free-running steps, ids and gamma bit-exact against the stored oracle trajectory."""
    wl = syn.workloads()["C1"]
    m, r = wl.model, wl.run
    om, g_dev, layers_dev = both_models(m, wl.seed, 0.02)
    prompt = syn.make_prompts(wl.seed, 1, r.prompt_lo, r.prompt_hi, m.vocab)[0].numpy()
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=1, max_seq_len=64 + r.steps * r.block_D + r.block_D, D=r.block_D, tau=r.tau)
    assert ctx.kernel_info == "generic-fp32"
    st, seqs = lockstep(ctx, om, [prompt], r.block_D, r.tau, r.steps, logit_tol=1e-4, conf_tol=1e-5)
    print("C1", st)
    gold = json.load(open(os.path.join(GOLD, "c1_trajectory.json")))
    assert [int(t) for t in seqs[0].tokens] == gold["final_tokens"]
    assert st.id_near_tie == 0 and st.gamma_near_tie == 0
    ctx.close()


@pytest.mark.parametrize("D,tau,paged", [(1, 0.5, False), (2, 0.9, True), (4, 0.8, False), (4, 0.8, True), (8, 0.6, True), (16, 0.3, False)])
def test_small_fp32_ragged_batch(D, tau, paged):
    """Ragged batch, several block sizes, both cache layouts, override and own commits alternating."""
    m = gpu_cfg()
    om, g_dev, layers_dev = both_models(m, seed=5, std=0.3)
    lens = [1, 2, 15, 16, 17, 33, 40]
    prompts = [syn.uniform_int(D, f"p{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    steps = 7
    ovr = syn.make_overrides(9, steps, len(lens), D, m.vocab)
    max_len = max(lens) + steps * D + D
    n_pages = sum((n + steps * D + 15) // 16 + 1 for n in lens)
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=len(lens), max_seq_len=max_len, D=D, tau=tau, paged=paged, n_pages=n_pages,
                      prefill_rows=64)
    st, _ = lockstep(ctx, om, prompts, D, tau, steps, logit_tol=1e-4, conf_tol=1e-5, overrides=ovr, max_len=max_len)
    print(f"D={D} paged={paged}", st)
    if D >= 4:
        assert max(st.gammas) > 1
    ctx.close()


@pytest.mark.parametrize("conf_fn,rule", [(1, 0), (0, 1), (1, 1)])
def test_confidence_and_rule_variants(conf_fn, rule):
    m = gpu_cfg(has_qkv_bias=False, n_q_heads=6, n_kv_heads=2, hidden=96, head_dim=64)
    om, g_dev, layers_dev = both_models(m, seed=6, std=0.3)
    prompts = [syn.uniform_int(3, f"q{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate([5, 9, 30])]
    tau = 0.02 if conf_fn == 1 else 0.2
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=3, max_seq_len=80, D=4, tau=tau, conf_fn=conf_fn, accept_rule=rule)
    st, _ = lockstep(ctx, om, prompts, 4, tau, 5, logit_tol=1e-4, conf_tol=1e-5, conf_fn=conf_fn, rule=rule)
    print(st)
    ctx.close()


def test_small_bf16_generic_kernels():
    """bf16 storage through the shape-generic kernels (head_dim 64 is not served by the matrix-core path)."""
    m = gpu_cfg(dtype="bf16", head_dim=64, hidden=128, n_q_heads=4, n_kv_heads=2)
    om, g_dev, layers_dev = both_models(m, seed=7, std=0.08)
    prompts = [syn.uniform_int(4, f"b{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate([3, 20, 37])]
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=3, max_seq_len=80, D=4, tau=0.1, paged=True, n_pages=20)
    st, _ = lockstep(ctx, om, prompts, 4, 0.1, 6, logit_tol=2e-2, conf_tol=2e-2, bf16=True)
    print(st)
    ctx.close()


def test_step_is_repeatable_and_batch_independent():
    """One, two and three sequences (8 to 24 rows): the same kernels, the same bits.  Batches beyond 32 rows: the test after this one."""
    m = gpu_cfg()
    om, g_dev, layers_dev = both_models(m, seed=8, std=0.3)
    prompts = [syn.uniform_int(5, f"r{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate([7, 21, 12])]
    D, V = 4, m.vocab
    outs = []
    for sel in ([0, 1, 2], [1], [2, 0]):
        ctx = gpu_context(m, g_dev, layers_dev, max_batch=3, max_seq_len=64, D=D, tau=0.05)
        ctx.prefill([prompts[i] for i in sel])
        B = len(sel)
        ids = torch.empty(B, D, dtype=torch.int32, device="cuda")
        cnt = torch.empty(B, dtype=torch.int32, device="cuda")
        logits = torch.empty(B * D, V, dtype=torch.float32, device="cuda")
        res = {}
        for t in range(3):
            ctx.decode_step(ids, cnt, None, logits)
            torch.cuda.synchronize()
            first = logits.clone()
            ctx.decode_step(ids, cnt, None, logits)          # repeated before commit: identical
            torch.cuda.synchronize()
            assert torch.equal(first, logits)
            for j, i in enumerate(sel):
                res[(i, t)] = logits.view(B, D, V)[j].cpu().clone()
            ctx.kv_commit()
        outs.append(res)
        ctx.close()
    for res in outs[1:]:
        for key, val in res.items():
            assert torch.equal(val, outs[0][key]), f"sequence {key[0]} step {key[1]} depends on its batch mates"


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_batches_on_both_sides_of_the_few_row_line(dtype):
    """Four sequences of D = 4 (32 rows) take the kernels for few rows, five (40) the separate ones: a sequence's results and cache entries agree to the order of the
    sums (bf16: to the roundings of the operands, each side within 2e-2 of exact), and alone or with three others, on one side, in every bit."""
    m = gpu_cfg(dtype=dtype, vocab=300)
    _, g_dev, layers_dev = both_models(m, seed=8, std=0.3 if dtype == "fp32" else 0.08)
    prompts = [syn.uniform_int(5, f"r{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate([7, 21, 12, 30, 18])]
    D, V, out = 4, m.vocab, []
    ovr = syn.make_overrides(15, 3, 5, D, V)
    for sel in ([0, 1, 2, 3, 4], [0, 1, 2, 3], [1]):
        B = len(sel)
        ctx = gpu_context(m, g_dev, layers_dev, max_batch=B, max_seq_len=64, D=D, tau=0.05)
        ctx.prefill([prompts[i] for i in sel])
        ids = torch.empty(B, D, dtype=torch.int32, device="cuda")
        cnt = torch.empty(B, dtype=torch.int32, device="cuda")
        logits = torch.empty(B, D, V, dtype=torch.float32, device="cuda")
        res = []
        for t in range(3):
            ctx.decode_step(ids, cnt, None, logits)
            torch.cuda.synchronize()
            res.append(logits[sel.index(1)].clone())
            ctx.kv_commit(ovr[0][t][sel].to(torch.int32).cuda().contiguous(), ovr[1][t][sel].to(torch.int32).cuda())
        n = int(ctx.get_lengths()[1][sel.index(1)])
        res += [x for layer in range(m.n_layers) for x in ctx.read_kv(layer, sel.index(1), 0, 0, n)]
        out.append(res)
        ctx.close()
    for few, alone, many in zip(out[1], out[2], out[0]):
        assert torch.equal(few, alone)
        assert (few - many).abs().max() <= (2e-5 if dtype == "fp32" else 4e-2) * many.abs().max()


def test_cache_contents_match_oracle_cache():
    m = gpu_cfg()
    om, g_dev, layers_dev = both_models(m, seed=10, std=0.3)
    prompts = [syn.uniform_int(6, f"k{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate([18, 5])]
    D = 4
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=2, max_seq_len=64, D=D, tau=0.05, paged=True, n_pages=12)
    st, seqs = lockstep(ctx, om, prompts, D, 0.05, 4, logit_tol=1e-4, conf_tol=1e-5)
    for b, s in enumerate(seqs):
        for layer in range(m.n_layers):
            for hk in range(m.n_kv_heads):
                k, v = ctx.read_kv(layer, b, hk, 0, s.c)
                for pos in range(s.c):
                    ko, vo = s.read_kv(layer, pos, hk)
                    assert np.max(np.abs(k[pos].numpy() - ko)) < 1e-4 * max(1.0, np.max(np.abs(ko)))
                    assert np.max(np.abs(v[pos].numpy() - vo)) < 1e-4 * max(1.0, np.max(np.abs(vo)))
    ctx.close()


def test_error_paths():
    from paper_2509_24007_amd import sdlm
    m = gpu_cfg()
    om, g_dev, layers_dev = both_models(m, seed=11, std=0.3)
    with pytest.raises(sdlm.SdlmError) as e:
        gpu_context(m, g_dev, layers_dev, max_batch=1, max_seq_len=32, D=17, tau=0.5)
    assert e.value.code == sdlm.EINVAL
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=2, max_seq_len=24, D=4, tau=0.5)
    ids = torch.empty(2, 4, dtype=torch.int32, device="cuda")
    cnt = torch.empty(2, dtype=torch.int32, device="cuda")
    with pytest.raises(sdlm.SdlmError) as e:
        ctx.decode_step(ids, cnt)
    assert e.value.code == sdlm.ESTATE
    with pytest.raises(sdlm.SdlmError) as e:
        ctx.prefill([[1, 2, 3], []])
    assert e.value.code == sdlm.EINVAL
    with pytest.raises(sdlm.SdlmError) as e:
        ctx.prefill([list(range(21))])                      # 21 + D > 24
    assert e.value.code == sdlm.ECAPACITY
    with pytest.raises(sdlm.SdlmError) as e:
        ctx.prefill([[1, 2, m.vocab]])
    assert e.value.code == sdlm.EINVAL
    ctx.prefill([[1, 2, 3], [4, 5]])
    with pytest.raises(sdlm.SdlmError) as e:
        ctx.kv_commit()
    assert e.value.code == sdlm.ESTATE
    four = torch.full((2,), 4, dtype=torch.int32, device="cuda")
    toks = torch.ones(2, 4, dtype=torch.int32, device="cuda")
    with pytest.raises(sdlm.SdlmError) as e:
        for _ in range(8):                                  # 3 + 4k tokens: capacity trips before any overflow
            ctx.decode_step(ids, cnt)
            ctx.kv_commit(toks, four)
    assert e.value.code == sdlm.ECAPACITY
    n, c = ctx.get_lengths()
    assert int(n.max()) + 4 > 24 and int(n.max()) <= 24
    # a clamped override count is reported
    ctx.prefill([[1, 2, 3]])
    ctx.decode_step(ids, cnt)
    ctx.kv_commit(toks, torch.full((2,), 9, dtype=torch.int32, device="cuda"))
    with pytest.raises(sdlm.SdlmError) as e:
        ctx.get_lengths()
    assert e.value.code == sdlm.EINVAL
    # an override token outside the vocabulary is replaced and reported
    ctx.prefill([[1, 2, 3]])
    ctx.decode_step(ids, cnt)
    bad = torch.full((2, 4), m.vocab + 5, dtype=torch.int32, device="cuda")
    ctx.kv_commit(bad, torch.ones(2, dtype=torch.int32, device="cuda"))
    with pytest.raises(sdlm.SdlmError) as e:
        ctx.get_lengths()
    assert e.value.code == sdlm.EINVAL
    ctx.decode_step(ids, cnt)                               # and the next step still runs on valid rows
    torch.cuda.synchronize()
    ctx.close()
    # paged pool too small for the prompts
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=2, max_seq_len=64, D=4, tau=0.5, paged=True, n_pages=2)
    with pytest.raises(sdlm.SdlmError) as e:
        ctx.prefill([list(range(20)), list(range(20))])
    assert e.value.code == sdlm.ECAPACITY
    ctx.prefill([list(range(14)), list(range(14))])
    with pytest.raises(sdlm.SdlmError) as e:
        for _ in range(4):
            ctx.decode_step(ids, cnt)
            ctx.kv_commit(toks, four)
    assert e.value.code == sdlm.ECAPACITY
    ctx.close()


@pytest.mark.parametrize("paged", [False, True])
def test_commit_at_the_capacity_edge(paged):
    """A step is admitted only if accepting all D tokens still fits (n + D <= max_seq_len), so a commit can never run
    out of positions or page-table entries on the device: with max_seq_len a multiple of the page size, a sequence
    that fills up exactly keeps every accepted token, reports no error, and the next step is refused on the host."""
    from paper_2509_24007_amd import sdlm
    m = gpu_cfg()
    om, g_dev, layers_dev = both_models(m, seed=13, std=0.3)
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=2, max_seq_len=64, D=4, tau=0.5, paged=paged, n_pages=8 if paged else 0)
    with pytest.raises(sdlm.SdlmError) as e:
        ctx.prefill([list(range(61)), [1, 2]])              # 61 + 4 > 64: all four tokens could not be kept
    assert e.value.code == sdlm.ECAPACITY
    prompts = [syn.uniform_int(13, "edge", 60, 0, m.vocab - 1).numpy(), np.array([3, 4], np.int32)]
    seqs = [orc.Seq(om, 64) for _ in prompts]
    for s, p in zip(seqs, prompts):
        s.prefill(p)
    ctx.prefill(prompts)
    ids = torch.empty(2, 4, dtype=torch.int32, device="cuda")
    cnt = torch.empty(2, dtype=torch.int32, device="cuda")
    logits = torch.empty(8, m.vocab, dtype=torch.float32, device="cuda")
    ctx.decode_step(ids, cnt, None, logits)
    toks = torch.tensor([[5, 6, 7, 8], [9, 10, 11, 12]], dtype=torch.int32, device="cuda")
    ctx.kv_commit(toks, torch.tensor([4, 1], dtype=torch.int32, device="cuda"))
    n, c = ctx.get_lengths()                                # no device-side error flag
    assert n.tolist() == [64, 3] and c.tolist() == [60, 2]
    with pytest.raises(sdlm.SdlmError) as e:
        ctx.decode_step(ids, cnt)                           # 64 + 4 > 64
    assert e.value.code == sdlm.ECAPACITY
    ctx.close()
    # the same two sequences with room for one more step: the four committed tokens are really there (the step after
    # the commit matches the oracle, which was fed the same tokens)
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=2, max_seq_len=80, D=4, tau=0.5, paged=paged, n_pages=10 if paged else 0)
    seqs = [orc.Seq(om, 80) for _ in prompts]
    for s, p in zip(seqs, prompts):
        s.prefill(p)
    ctx.prefill(prompts)
    ctx.decode_step(ids, cnt)
    for s in seqs:
        s.step(4, 0.5)
    ctx.kv_commit(toks, torch.tensor([4, 1], dtype=torch.int32, device="cuda"))
    assert seqs[0].commit([5, 6, 7, 8], 4) == 0 and seqs[1].commit([9], 1) == 0
    ctx.decode_step(ids, cnt, None, logits)
    torch.cuda.synchronize()
    z = logits.cpu().numpy().reshape(2, 4, -1)
    for b in range(2):
        lo, io, _, _ = seqs[b].step(4, 0.5)
        assert np.max(np.abs(z[b] - lo)) <= 1e-4 * np.max(np.abs(lo))
    ctx.close()


@pytest.mark.parametrize("dtype,hd", [("fp32", 32), ("bf16", 128)])
def test_nan_logits_still_give_valid_ids(dtype, hd):
    """Non-finite weights must not turn into out-of-range token ids (they would index the embedding table)."""
    m = gpu_cfg(dtype=dtype, head_dim=hd, hidden=128, ffn=128, n_q_heads=2, n_kv_heads=1) if dtype == "fp32" else mfma_cfg()
    om, g_dev, layers_dev = both_models(m, seed=12, std=0.05)
    g_dev = dict(g_dev)
    g_dev["lm_head"] = torch.full_like(g_dev["lm_head"], float("nan"))
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=2, max_seq_len=64, D=4, tau=0.5)
    ctx.prefill([[1, 2, 3], [4]])
    ids = torch.empty(2, 4, dtype=torch.int32, device="cuda")
    cnt = torch.empty(2, dtype=torch.int32, device="cuda")
    for _ in range(3):
        ctx.decode_step(ids, cnt)
        ctx.kv_commit()
    torch.cuda.synchronize()
    assert int(ids.min()) >= 0 and int(ids.max()) < m.vocab
    assert int(cnt.min()) >= 1 and int(cnt.max()) <= 4
    ctx.close()


def test_generator_is_identical_on_cpu_and_gpu():
    a = syn.normal(3, "dev", (1000, 33), 0.02, torch.bfloat16, "cpu")
    b = syn.normal(3, "dev", (1000, 33), 0.02, torch.bfloat16, "cuda")
    assert torch.equal(a, b.cpu())
    assert torch.equal(syn.uniform_int(3, "u", 5000, 0, 151935), syn.uniform_int(3, "u", 5000, 0, 151935, device="cuda").cpu())


# ------------------------------------------------------------------ bf16 matrix-core path (head_dim 128)

def mfma_cfg(**kw):
    base = dict(n_layers=2, hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=128, ffn=512, vocab=2048, dtype="bf16",
                rope_theta=1.0e6, has_qkv_bias=True)
    base.update(kw)
    return syn.ModelCfg(**base)


@pytest.mark.parametrize("name,kw,lens,D,tau,paged", [
    ("g2", {}, [1, 9, 40, 100], 4, 0.6, True),
    ("g7-ragged-vocab", dict(n_q_heads=14, n_kv_heads=2, vocab=1000, ffn=320), [3, 17, 33, 64, 70], 4, 0.6, True),
    ("g8-D8-two-groups", dict(n_q_heads=16, n_kv_heads=2, hidden=512), [5, 130, 300], 8, 0.5, False),
    ("g6-D4-batch1-long", dict(n_q_heads=12, n_kv_heads=2, hidden=384, ffn=1024), [700], 4, 0.6, False),
    ("g4-batch20-128-row-tiles", dict(n_q_heads=8, n_kv_heads=2, vocab=4096 + 160), [3 + 7 * i for i in range(20)], 4, 0.6, True),
    ("g5-D16", dict(n_q_heads=10, n_kv_heads=2, hidden=320, ffn=640, has_qkv_bias=False), [2, 50], 16, 0.3, True),
    ("g4-batch36-256-row-gate-up-tile", dict(n_q_heads=8, n_kv_heads=2, hidden=256, ffn=24576), [3 + 2 * i for i in range(36)], 4, 0.6, True),
])
def test_bf16_mfma_path(name, kw, lens, D, tau, paged):
    """The bf16 product path: MFMA GEMMs, MFMA block-masked attention (split KV), fused LM-head reduction."""
    m = mfma_cfg(**kw)
    om, g_dev, layers_dev = both_models(m, seed=21, std=0.05)
    prompts = [syn.uniform_int(D, f"{name}{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    steps = 6
    ovr = syn.make_overrides(13, steps, len(lens), D, m.vocab)
    max_len = max(lens) + steps * D + D
    n_pages = sum((n + steps * D + 15) // 16 + 1 for n in lens)
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=len(lens), max_seq_len=max_len, D=D, tau=tau, paged=paged, n_pages=n_pages,
                      prefill_rows=128)
    assert ctx.kernel_info == "mfma-bf16"
    st, _ = lockstep(ctx, om, prompts, D, tau, steps, logit_tol=2e-2, conf_tol=1e-3, overrides=ovr, bf16=True, max_len=max_len)
    print(name, st)
    ctx.close()


def test_bf16_mfma_entropy_confidence():
    m = mfma_cfg()
    om, g_dev, layers_dev = both_models(m, seed=22, std=0.05)
    prompts = [syn.uniform_int(1, f"e{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate([12, 31])]
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=2, max_seq_len=80, D=4, tau=0.05, conf_fn=1)
    st, _ = lockstep(ctx, om, prompts, 4, 0.05, 4, logit_tol=2e-2, conf_tol=1e-3, conf_fn=1, bf16=True)
    print(st)
    ctx.close()


# ------------------------------------------------------------------ self-speculative verification (Sec. 3.4, Eq. 10)
@pytest.mark.parametrize("D,rule,paged", [(2, 0, False), (3, 1, True), (4, 0, True), (4, 1, False), (5, 0, False), (6, 0, True), (8, 0, False),
                                          (9, 1, False), (10, 0, True), (12, 1, False), (16, 0, True)])
def test_verify_small_fp32(D, rule, paged):
    """Second pass of a self-speculative step against the oracle's: logits of every verification input, ytilde,
    gamma_verify bit-exact, and the verified count is what an argument-less commit publishes.  The causal rows of the
    speculative tokens are computed once per sequence; D <= 4: all rows of a sequence share one staging tile, D >= 5: the
    causal rows and every input's block have tiles of their own and a block row reads two of them."""
    m = gpu_cfg()
    om, g_dev, layers_dev = both_models(m, seed=6, std=0.3)
    lens = [1, 2, 15, 16, 17, 33]
    prompts = [syn.uniform_int(D, f"v{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    steps = 5
    ovr = syn.make_overrides(10, steps, len(lens), D, m.vocab)
    max_len = max(lens) + steps * D + D
    n_pages = sum((n + steps * D + 15) // 16 + 1 for n in lens)
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=len(lens), max_seq_len=max_len, D=D, tau=0.5, paged=paged, n_pages=n_pages,
                      prefill_rows=64)
    st, _ = lockstep(ctx, om, prompts, D, 0.5, steps, logit_tol=1e-4, conf_tol=1e-5, overrides=ovr, max_len=max_len,
                     verify_rule=rule)
    print(f"verify D={D} rule={rule}", st, "verify rows", st.verify_rows, "gammas", np.bincount(st.verify_gammas))
    assert st.verify_rows == steps * len(lens) * (D - 1) and st.verify_skipped == 0 and st.verify_near_tie == 0
    ctx.close()


@pytest.mark.parametrize("paged,prefill_rows", [(True, 256), (False, 4096)])
def test_long_prefill_cache_matches_oracle_cache_bf16(paged, prefill_rows):
    """Prefill of long prompts on the matrix-core path (several passes when prefill_rows is below the prompt length,
    several KV chunks per attention work item, ragged last groups): every cached K and V vector of every layer, kv head
    and position against the oracle's cache, which by its pins holds the K/V of the real tokens under causal attention
    (Sec. 3.3: every block sees the real tokens before it causally).  The layers' inputs differ by bf16 rounding, so
    the comparison is per vector, relative to the vector's largest entry."""
    m = mfma_cfg(n_layers=3, n_q_heads=14, n_kv_heads=2, hidden=256, ffn=512)
    om, g_dev, layers_dev = both_models(m, seed=31, std=0.05)
    lens = [700, 1, 333, 1025]
    prompts = [syn.uniform_int(31, f"lp{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    D = 4
    n_pages = sum((n + 2 * D + 15) // 16 + 1 for n in lens)
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=len(lens), max_seq_len=max(lens) + 2 * D, D=D, tau=0.5, paged=paged,
                      n_pages=n_pages if paged else 0, prefill_rows=prefill_rows)
    assert ctx.kernel_info == "mfma-bf16"
    ctx.prefill(prompts)
    n, c = ctx.get_lengths()
    assert n.tolist() == lens and c.tolist() == lens
    worst_k = worst_v = 0.0
    for b, p in enumerate(prompts):
        s = orc.Seq(om, len(p) + 2 * D)
        s.prefill(p)
        for layer in range(m.n_layers):
            for hk in range(m.n_kv_heads):
                k, v = ctx.read_kv(layer, b, hk, 0, len(p))
                k, v = k.numpy().astype(np.float64), v.numpy().astype(np.float64)
                for pos in range(len(p)):
                    ko, vo = s.read_kv(layer, pos, hk)
                    worst_k = max(worst_k, float(np.max(np.abs(k[pos] - ko)) / np.max(np.abs(ko))))
                    worst_v = max(worst_v, float(np.max(np.abs(v[pos] - vo)) / np.max(np.abs(vo))))
    print(f"long prefill paged={paged} rows/pass={prefill_rows}: worst relative K error {worst_k:.3e}, V {worst_v:.3e}")
    assert worst_k <= 2e-2 and worst_v <= 2e-2
    ctx.close()


@pytest.mark.parametrize("name,lens", [
    ("small-step", [9, 33]),                                   # at most 32 rows per step: QKV, RoPE and K/V placement are one launch
    ("larger-step", [3 + 5 * i for i in range(9)]),            # 72 rows: projection, then the RoPE + K/V placement kernel
])
def test_decode_cache_matches_oracle_cache_bf16(name, lens):
    """K/V written by decode steps on the matrix-core path: after several steps with forced acceptance counts, every cached K
    and V vector (prompt positions and the positions of the committed tokens, whose K/V came from the pending rows of
    later steps) against the oracle's clean cache (Sec. 3.3: only real tokens under causal attention are ever cached).
    Both QKV paths are covered: the fused launch of small steps and the separate kernels of larger ones."""
    m = mfma_cfg(n_q_heads=6, n_kv_heads=2, hidden=256, ffn=512)
    om, g_dev, layers_dev = both_models(m, seed=41, std=0.05)
    D, steps = 4, 5
    prompts = [syn.uniform_int(41, f"dc{name}{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    ovr = syn.make_overrides(17, steps, len(lens), D, m.vocab)   # forced tokens and counts on some steps: pending runs of every length
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=len(lens), max_seq_len=max(lens) + (steps + 2) * D, D=D, tau=0.5, paged=True,
                      n_pages=sum((n + (steps + 2) * D + 15) // 16 + 1 for n in lens))
    assert ctx.kernel_info == "mfma-bf16"
    st, seqs = lockstep(ctx, om, prompts, D, 0.5, steps, logit_tol=2e-2, conf_tol=1e-5, overrides=ovr, bf16=True)
    worst_k = worst_v = 0.0
    grown = 0
    for b, s in enumerate(seqs):
        grown += s.c - len(prompts[b])
        for layer in range(m.n_layers):
            for hk in range(m.n_kv_heads):
                k, v = ctx.read_kv(layer, b, hk, 0, s.c)
                k, v = k.numpy().astype(np.float64), v.numpy().astype(np.float64)
                for pos in range(s.c):
                    ko, vo = s.read_kv(layer, pos, hk)
                    worst_k = max(worst_k, float(np.max(np.abs(k[pos] - ko)) / np.max(np.abs(ko))))
                    worst_v = max(worst_v, float(np.max(np.abs(v[pos] - vo)) / np.max(np.abs(vo))))
    print(f"decode cache {name}: {grown} positions written by pending rows, worst relative K error {worst_k:.3e}, V {worst_v:.3e}")
    assert grown >= steps * len(lens) - len(lens)   # every step but the last one's commit has left its tokens in the cache
    assert worst_k <= 2e-2 and worst_v <= 2e-2
    ctx.close()


def test_verify_position_independent_model_accepts_whole_block():
    """All-zero weights: every logit row is constant, arg-max is token 0 everywhere, so every position verifies."""
    m = gpu_cfg()
    om, g_dev, layers_dev = both_models(m, seed=6, std=0.0)
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=2, max_seq_len=64, D=4, tau=2.0)
    ctx.prefill([np.array([4, 2, 7], dtype=np.int32), np.array([1], dtype=np.int32)])
    ids = torch.empty(2, 4, dtype=torch.int32, device="cuda")
    cnt = torch.empty(2, dtype=torch.int32, device="cuda")
    vid = torch.empty(2, 4, dtype=torch.int32, device="cuda")
    vc = torch.empty(2, dtype=torch.int32, device="cuda")
    ctx.decode_step(ids, cnt)
    ctx.verify_step(0, vid, vc)
    torch.cuda.synchronize()
    assert cnt.tolist() == [1, 1] and vc.tolist() == [4, 4]
    assert ids.cpu().eq(0).all() and vid.cpu().eq(0).all()
    ctx.kv_commit()
    n, c = ctx.get_lengths()
    assert n.tolist() == [3 + 4, 1 + 4]
    ctx.close()


def test_phase_timers_count_launches_and_sample():
    """The per-phase event timers report one launch per layer and step for a per-layer phase, every n-th of them when
    sampling, and the sampled steps produce the same tokens as the untimed ones."""
    m = mfma_cfg(n_layers=3)
    om, g_dev, layers_dev = both_models(m, seed=8, std=0.05)
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=2, max_seq_len=64, D=4, tau=0.5)
    prompts = [np.array([1, 2, 3], dtype=np.int32), np.array([4, 5], dtype=np.int32)]
    ids = torch.empty(3, 2, 4, dtype=torch.int32, device="cuda")
    cnt = torch.empty(3, 2, dtype=torch.int32, device="cuda")
    from paper_2509_24007_amd.sdlm import SdlmError
    for mode, (every, steps) in enumerate([(1, 2), (2, 3), (7, 2)]):
        ctx.prefill(prompts)
        ctx.profile(["gateup", "lmhead"], every=every)
        for _ in range(steps):
            ctx.decode_step(ids[mode], cnt[mode])
        got = ctx.profile_read()
        ctx.profile(None)
        assert got["gateup"][1] == -(-3 * steps // every) and got["lmhead"][1] == -(-steps // every)
        assert got["gateup"][0] > 0.0 and got["qkv"] == (0.0, 0)
    torch.cuda.synchronize()
    assert ids[0].eq(ids[1]).all() and ids[0].eq(ids[2]).all() and cnt[0].eq(cnt[1]).all() and cnt[0].eq(cnt[2]).all()
    with pytest.raises(SdlmError):
        ctx.profile(["gateup"], every=0)
    ctx.close()


def test_verify_error_paths():
    m = gpu_cfg()
    om, g_dev, layers_dev = both_models(m, seed=6, std=0.3)
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=1, max_seq_len=64, D=4, tau=0.5)
    ctx.prefill([np.array([1, 2, 3], dtype=np.int32)])
    from paper_2509_24007_amd.sdlm import SdlmError
    with pytest.raises(SdlmError):
        ctx.verify_step(0)              # no step yet
    ids = torch.empty(1, 4, dtype=torch.int32, device="cuda")
    cnt = torch.empty(1, dtype=torch.int32, device="cuda")
    ctx.decode_step(ids, cnt)
    with pytest.raises(SdlmError):
        ctx.verify_step(2)              # unknown rule
    ctx.verify_step(0)
    ctx.verify_step(1)                  # may be repeated before the commit
    ctx.kv_commit()
    with pytest.raises(SdlmError):
        ctx.verify_step(0)              # the step has been committed
    ctx.close()


@pytest.mark.parametrize("name,kw,lens,D", [
    ("vg2", {}, [1, 9, 40, 100], 4),
    ("vg7", dict(n_q_heads=14, n_kv_heads=2, vocab=1000, ffn=320), [3, 17, 33, 64, 70], 4),
    ("vg8-D8-two-groups-per-input", dict(n_q_heads=16, n_kv_heads=2, hidden=512), [5, 130, 300], 8),
    ("vg16-four-groups-across-inputs", dict(n_q_heads=16, n_kv_heads=1, hidden=256), [2, 31, 90], 4),
    ("vg4-D3", dict(n_q_heads=8, n_kv_heads=2), [7, 16, 49], 3),
    ("vg3-D5-two-staging-tiles", dict(n_q_heads=6, n_kv_heads=2), [4, 40], 5),
    ("vg7-D9", dict(n_q_heads=14, n_kv_heads=2, vocab=1000, ffn=320), [3, 70], 9),
    ("vg4-D16", dict(n_q_heads=8, n_kv_heads=2), [1, 33, 200], 16),
])
def test_verify_bf16_mfma(name, kw, lens, D):
    m = mfma_cfg(**kw)
    om, g_dev, layers_dev = both_models(m, seed=21, std=0.05)
    prompts = [syn.uniform_int(D, f"{name}{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    steps = 4
    max_len = max(lens) + steps * D + D
    n_pages = sum((n + steps * D + 15) // 16 + 1 for n in lens)
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=len(lens), max_seq_len=max_len, D=D, tau=0.6, paged=True, n_pages=n_pages,
                      prefill_rows=128)
    assert ctx.kernel_info == "mfma-bf16"
    st, _ = lockstep(ctx, om, prompts, D, 0.6, steps, logit_tol=2e-2, conf_tol=1e-3, bf16=True, max_len=max_len, verify_rule=0)
    print(name, st, "verify rows", st.verify_rows, "skipped", st.verify_skipped, "near ties", st.verify_near_tie)
    assert st.verify_rows > 0
    ctx.close()


# ------------------------------------------------------------------ causal attention inside the block (Sec. 4.4 ablation)
@pytest.mark.parametrize("D,paged,verify", [(4, False, None), (8, True, None), (4, True, 0)])
def test_block_causal_small_fp32(D, paged, verify):
    m = gpu_cfg(block_causal=True)
    om, g_dev, layers_dev = both_models(m, seed=7, std=0.3)
    assert om.cfg.block_causal == 1
    lens = [1, 5, 16, 31]
    prompts = [syn.uniform_int(D, f"bc{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    steps = 5
    ovr = syn.make_overrides(11, steps, len(lens), D, m.vocab)
    max_len = max(lens) + steps * D + D
    n_pages = sum((n + steps * D + 15) // 16 + 1 for n in lens)
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=len(lens), max_seq_len=max_len, D=D, tau=0.6, paged=paged, n_pages=n_pages,
                      prefill_rows=64)
    st, _ = lockstep(ctx, om, prompts, D, 0.6, steps, logit_tol=1e-4, conf_tol=1e-5, overrides=ovr, max_len=max_len,
                     verify_rule=verify)
    print(f"block-causal D={D}", st)
    assert st.id_near_tie == 0
    ctx.close()


def test_block_causal_bf16_mfma():
    m = mfma_cfg(block_causal=True)
    om, g_dev, layers_dev = both_models(m, seed=21, std=0.05)
    lens = [1, 9, 40, 100]
    prompts = [syn.uniform_int(4, f"bcm{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    steps = 4
    max_len = max(lens) + steps * 4 + 4
    n_pages = sum((n + steps * 4 + 15) // 16 + 1 for n in lens)
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=len(lens), max_seq_len=max_len, D=4, tau=0.6, paged=True, n_pages=n_pages,
                      prefill_rows=128)
    assert ctx.kernel_info == "mfma-bf16"
    st, _ = lockstep(ctx, om, prompts, 4, 0.6, steps, logit_tol=2e-2, conf_tol=1e-3, bf16=True, max_len=max_len, verify_rule=0)
    print("block-causal mfma", st)
    ctx.close()


# ------------------------------------------------------------------ HIP-graph replay of the step
@pytest.mark.parametrize("kind", ["fp32", "mfma"])
def test_graph_replay_matches_oracle_and_eager(kind):
    """Every replay is checked against the oracle, with the library's eager commit kernels (own and override) and host
    synchronisations between replays; then a replayed and an eager context are compared bit for bit."""
    if kind == "fp32":
        m, std, tol, ctol, bf = gpu_cfg(), 0.3, 1e-4, 1e-5, False
    else:
        m, std, tol, ctol, bf = mfma_cfg(), 0.05, 2e-2, 1e-3, True
    om, g_dev, layers_dev = both_models(m, seed=8, std=std)
    lens = [1, 7, 16, 33, 40]
    D, tau, steps = 4, 0.6, 8
    prompts = [syn.uniform_int(3, f"gr{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    ovr = syn.make_overrides(12, steps, len(lens), D, m.vocab)
    max_len = max(lens) + steps * D + D
    n_pages = sum((n + steps * D + 15) // 16 + 1 for n in lens)
    side = torch.cuda.Stream()
    kw = dict(max_batch=len(lens), max_seq_len=max_len, D=D, tau=tau, paged=True, n_pages=n_pages, prefill_rows=64)
    ctx = gpu_context(m, g_dev, layers_dev, stream=side, **kw)
    ctx.graph(True)
    st, _ = lockstep(ctx, om, prompts, D, tau, steps, logit_tol=tol, conf_tol=ctol, overrides=ovr, bf16=bf, max_len=max_len)
    print("graph", kind, st)
    # replayed vs eager, same inputs, fresh contexts: identical bits
    outs = []
    for use_graph in (True, False):
        c2 = gpu_context(m, g_dev, layers_dev, stream=side, **kw)
        if use_graph:
            c2.graph(True)
        c2.prefill(prompts)
        ids = torch.empty(steps, len(lens), D, dtype=torch.int32, device="cuda")
        cnt = torch.empty(steps, len(lens), dtype=torch.int32, device="cuda")
        conf = torch.empty(len(lens), D, dtype=torch.float32, device="cuda")
        logits = torch.empty(len(lens) * D, m.vocab, dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        trace = []
        for t in range(steps):
            c2.decode_step(ids[t], cnt[t], conf, logits) if t % 3 else c2.decode_step(ids[t], cnt[t])   # the outputs change: re-capture
            torch.cuda.synchronize()
            trace.append((conf.clone(), logits.clone()) if t % 3 else None)
            c2.kv_commit()
        torch.cuda.synchronize()
        outs.append((ids.cpu(), cnt.cpu(), trace))
        c2.close()
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    for a, b in zip(outs[0][2], outs[1][2]):
        if a is not None:
            assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    ctx.close()


@pytest.mark.parametrize("start", [230, 490])
def test_graph_replay_is_eager_bit_for_bit_as_contexts_grow(start):
    """A context that holds far more than its sequences: replayed and eager steps agree in every bit before, at and after the lengths at which the
    attention's launches change (256 keys: teams of one workgroup; 512: the merge for more than eight chunks)."""
    m = mfma_cfg()
    _, g_dev, layers_dev = both_models(m, seed=18, std=0.05)
    D, steps = 8, 6
    prompts = [syn.uniform_int(18, f"gg{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate([start, 33])]
    ovr = syn.make_overrides(18, steps, 2, D, m.vocab)[0].to(torch.int32).cuda()
    side = torch.cuda.Stream()
    out = []
    for use_graph in (True, False):
        ctx = gpu_context(m, g_dev, layers_dev, stream=side, max_batch=2, max_seq_len=900, D=D, tau=0.5)
        ctx.graph(use_graph)
        ctx.prefill(prompts)
        ids = torch.empty(2, D, dtype=torch.int32, device="cuda")
        cnt = torch.empty(2, dtype=torch.int32, device="cuda")
        logits = torch.empty(2 * D, m.vocab, dtype=torch.float32, device="cuda")
        for t in range(steps):
            for _ in range(2):                           # the second call replays what the first one captured
                ctx.decode_step(ids, cnt, None, logits)
                torch.cuda.synchronize()
                out.append(logits.clone())
            ctx.kv_commit(ovr[t].contiguous(), torch.full((2,), D, dtype=torch.int32, device="cuda"))
        assert ctx.get_lengths()[0].tolist() == [start + steps * D, 33 + steps * D]
        ctx.close()
    for t, (a, b) in enumerate(zip(out[:2 * steps], out[2 * steps:])):
        assert torch.equal(a, b), f"step {t // 2}: replay and eager differ by {(a - b).abs().max().item():.3e}"


@pytest.mark.parametrize("static", [False, True])
def test_step_in_a_callers_graph_at_any_length(static):
    """A step that the caller records into a graph of its own at a short context is right at every length the context can hold: the attention's form for short
    contexts (at most 256 keys; its page numbers ride in 64 lanes, 1024 keys) must not be baked into it.  The graph serves other prompts of the same batch: 1300 tokens, where its
    launches are those of an eager step and so its bits, and again a short one, where only the order of the sums differs."""
    m = mfma_cfg()
    _, g_dev, layers_dev = both_models(m, seed=18, std=0.05)
    D = 8
    side = torch.cuda.Stream()
    ctx = gpu_context(m, g_dev, layers_dev, stream=side, max_batch=2, max_seq_len=1400, D=D, tau=0.5)
    ids = torch.empty(2, D, dtype=torch.int32, device="cuda")
    cnt = torch.empty(2, dtype=torch.int32, device="cuda")
    logits = torch.empty(2 * D, m.vocab, dtype=torch.float32, device="cuda")

    def fresh(n):
        ctx.prefill([syn.uniform_int(18, f"cg{n}{i}", k, 0, m.vocab - 1).numpy() for i, k in enumerate([n, 33])])
        ctx.decode_step(ids, cnt, None, logits, static_scratch=static)
        torch.cuda.synchronize()
        return logits.clone()

    eager = fresh(200)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side, capture_error_mode="thread_local"):
        ctx.decode_step(ids, cnt, None, logits, static_scratch=static)
    for n in (200, 1300, 200):
        eager = fresh(n)
        for _ in range(2):
            logits.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            err = ((logits - eager).abs().amax(1) / eager.abs().amax(1)).max().item()
            print("static" if static else "workspace", n, err)
            assert torch.equal(logits, eager) if n == 1300 else err <= 2e-2, (n, err)   # (the bar of the bf16 path)
    ctx.close()


def test_eager_steps_behind_a_callers_graph_that_commits():
    """A caller's graph of a step and its commit moves the lengths where the host does not see it; an eager step behind it is still that of the lengths there are."""
    m = mfma_cfg()
    _, g_dev, layers_dev = both_models(m, seed=18, std=0.05)
    D, start, steps = 16, 200, 62
    ovr = syn.make_overrides(19, 2, 1, D, m.vocab)[0][0].to(torch.int32).cuda().contiguous()
    full = torch.full((1,), D, dtype=torch.int32, device="cuda")
    prompt = [syn.uniform_int(18, "cc", start, 0, m.vocab - 1).numpy()]
    side = torch.cuda.Stream()
    out = []
    for replayed in (False, True):
        ctx = gpu_context(m, g_dev, layers_dev, stream=side, max_batch=1, max_seq_len=1300, D=D, tau=0.5)
        ids = torch.empty(1, D, dtype=torch.int32, device="cuda")
        cnt = torch.empty(1, dtype=torch.int32, device="cuda")
        logits = torch.empty(D, m.vocab, dtype=torch.float32, device="cuda")
        ctx.prefill(prompt)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        if replayed:
            with torch.cuda.graph(graph, stream=side, capture_error_mode="thread_local"):
                ctx.decode_step(ids, cnt)
                ctx.kv_commit(ovr, full)
        for _ in range(steps):
            if replayed:
                graph.replay()
            else:
                ctx.decode_step(ids, cnt)
                ctx.kv_commit(ovr, full)
            torch.cuda.synchronize()
        ctx.decode_step(ids, cnt, None, logits)
        torch.cuda.synchronize()
        out.append(logits.clone())
        assert ctx.get_lengths()[0].tolist() == [start + steps * D]
        ctx.close()
    err = ((out[1] - out[0]).abs().amax(1) / out[0].abs().amax(1)).max().item()
    print("eager behind a replayed commit", err)
    assert err <= 2e-2, err   # the cache is written by steps in another order of the sums (the bar of the bf16 path)


def test_graph_needs_a_real_stream():
    m = gpu_cfg()
    om, g_dev, layers_dev = both_models(m, seed=8, std=0.3)
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=1, max_seq_len=32, D=2, tau=0.5)
    from paper_2509_24007_amd.sdlm import SdlmError
    if ctx.stream.cuda_stream == 0:
        with pytest.raises(SdlmError):
            ctx.graph(True)
    ctx.graph(False)
    ctx.close()


def test_mfma_row_blocks_beyond_the_sure_ones():
    """Every sequence is forced to accept D tokens, so the next step has the maximum B*2D rows: the row blocks the
    launch lists last (those that may be empty) all hold rows.  Alternating with single-token commits exercises the
    ragged and the empty case of the same launch shape."""
    m = mfma_cfg(n_q_heads=8, n_kv_heads=2)
    om, g_dev, layers_dev = both_models(m, seed=21, std=0.05)
    B, D, steps = 24, 4, 6
    lens = [3 + 5 * i for i in range(B)]
    prompts = [syn.uniform_int(4, f"rb{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    ids, cnt = syn.make_overrides(14, steps, B, D, m.vocab)
    cnt = cnt.clone()
    for t in range(steps):
        cnt[t] = D if (t // 2) % 2 == 0 else 1       # lockstep applies the overrides on odd steps
    max_len = max(lens) + steps * D + D
    n_pages = sum((n + steps * D + 15) // 16 + 1 for n in lens)
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=B, max_seq_len=max_len, D=D, tau=0.6, paged=True, n_pages=n_pages,
                      prefill_rows=128)
    assert ctx.kernel_info == "mfma-bf16"
    st, _ = lockstep(ctx, om, prompts, D, 0.6, steps, logit_tol=2e-2, conf_tol=1e-3, overrides=(ids, cnt), bf16=True, max_len=max_len)
    print("row blocks", st)
    ctx.close()


@pytest.mark.parametrize("B,D,hidden,ffn", [(1, 1, 128, 192), (1, 4, 320, 576), (3, 4, 448, 1088), (4, 4, 1088, 320), (2, 8, 192, 2112)])
def test_bf16_gate_up_of_at_most_32_rows(B, D, hidden, ffn):
    """Steps of at most 32 rows (B * 2D <= 32) take the gate/up kernel that splits k over the wavefronts of a workgroup:
    k extents whose per-wavefront share is shorter than, equal to and longer than the two register sets, not a multiple
    of a set, and row counts from 1 to the full 32."""
    m = mfma_cfg(n_q_heads=4, n_kv_heads=2, hidden=hidden, ffn=ffn, vocab=1000, has_qkv_bias=True)
    # (wide layers with weights of std 0.05 saturate the activations: bf16 noise alone then passes the logit bound, in
    # either gate/up kernel)
    om, g_dev, layers_dev = both_models(m, seed=70 + B + D, std=0.05 if hidden < 1000 else 0.03)
    lens = [5 + 7 * i for i in range(B)]
    prompts = [syn.uniform_int(5, f"sk{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    steps = 4
    ids, cnt = syn.make_overrides(21, steps, B, D, m.vocab)
    cnt = cnt.clone()
    cnt[1] = D                                       # the step after a full commit has B * 2D rows
    max_len = max(lens) + steps * D + D
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=B, max_seq_len=max_len, D=D, tau=0.5)
    assert ctx.kernel_info == "mfma-bf16"
    st, _ = lockstep(ctx, om, prompts, D, 0.5, steps, logit_tol=2e-2, conf_tol=1e-3, overrides=(ids, cnt), bf16=True, max_len=max_len)
    assert st.step_rows[2] == B * 2 * D
    print("gate/up <= 32 rows", (B, D, hidden, ffn), st)
    ctx.close()


@pytest.mark.parametrize("B,D,hidden,heads", [(64, 8, 128, 12), (66, 8, 128, 12), (35, 8, 1600, 16), (46, 8, 1600, 16)])
def test_bf16_qkv_of_many_rows(B, D, hidden, heads):
    """Steps of 280 to 1056 rows on both sides of the fused QKV launch's last lines: 9 certain 64-row blocks by 64 columns (576 workgroups) and 10 of them, 5 by 80 (400) and 7;
    blocks that hold rows only after a full commit."""
    m = mfma_cfg(n_layers=2, n_q_heads=heads, n_kv_heads=2, hidden=hidden, ffn=64, vocab=100, has_qkv_bias=True)
    om, g_dev, layers_dev = both_models(m, seed=190 + B, std=0.03)
    prompts = [syn.uniform_int(8, f"mr{i}", 2 + i % 9, 0, m.vocab - 1).numpy() for i in range(B)]
    ids, cnt = syn.make_overrides(29, 3, B, D, m.vocab)
    cnt = cnt.clone()
    cnt[1] = D                                       # the step after a full commit has B * 2D rows
    max_len = max(len(p) for p in prompts) + 4 * D
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=B, max_seq_len=max_len, D=D, tau=0.5)
    assert ctx.kernel_info == "mfma-bf16"
    st, _ = lockstep(ctx, om, prompts, D, 0.5, 3, logit_tol=2e-2, conf_tol=1e-3, overrides=(ids, cnt), bf16=True, max_len=max_len)
    assert st.step_rows[0] == B * D and st.step_rows[2] == B * 2 * D
    print("qkv of many rows", (B, D, hidden, heads), st)
    ctx.close()


@pytest.mark.parametrize("lens,D,heads,kv,paged", [([1, 16, 17, 240], 4, 4, 2, False), ([31, 112, 129, 230, 2], 3, 6, 1, True), ([97], 16, 2, 2, True), ([244], 4, 12, 2, False)])
def test_bf16_attention_of_short_contexts(lens, D, heads, kv, paged):
    """Contexts of at most 256 keys: four teams of one workgroup stream the cache and merge in LDS.  Teams without a tile, odd tile counts, staging tile alone in
    its pair and beside a cache tile, several row groups a sequence; the last of the steps pass 256 keys, where the chunks are workgroups again."""
    m = mfma_cfg(n_layers=2, n_q_heads=heads, n_kv_heads=kv, hidden=256, ffn=320, vocab=300, has_qkv_bias=True)
    om, g_dev, layers_dev = both_models(m, seed=181, std=0.05)
    prompts = [syn.uniform_int(7, f"sc{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    steps, B = 5, len(lens)
    ids, cnt = syn.make_overrides(28, steps, B, D, m.vocab)
    max_len = max(lens) + (steps + 1) * D
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=B, max_seq_len=max(max_len, 300), D=D, tau=0.5, paged=paged, n_pages=sum((n + (steps + 1) * D + 15) // 16 for n in lens) if paged else 0)
    assert ctx.kernel_info == "mfma-bf16"
    st, _ = lockstep(ctx, om, prompts, D, 0.5, steps, logit_tol=2e-2, conf_tol=1e-3, overrides=(ids, cnt), bf16=True, max_len=max(max_len, 300), verify_rule=0 if 2 <= D <= 4 else None)
    print("short contexts", (lens, D, heads, kv, paged), st)
    ctx.close()


@pytest.mark.parametrize("B,D,hidden,ffn,heads", [(1, 1, 64, 64, 1), (1, 8, 192, 1024, 4), (2, 4, 576, 4160, 6), (1, 9, 1088, 8256, 10), (4, 2, 128, 9216, 8)])
def test_bf16_products_of_few_rows(B, D, hidden, ffn, heads):
    """The weight streams of steps of at most 16 rows (and QKV up to 32): k extents that leave wavefronts without a k step, that end
    inside a register set and that take several; one k range and up to sixteen split ones; row counts on both sides of 16."""
    m = mfma_cfg(n_layers=2, n_q_heads=heads, n_kv_heads=1 if heads == 1 else 2, hidden=hidden, ffn=ffn, vocab=1000, has_qkv_bias=True)
    om, g_dev, layers_dev = both_models(m, seed=100 + B + D, std=0.03)
    prompts = [syn.uniform_int(5, f"fr{i}", 3 + 14 * i, 0, m.vocab - 1).numpy() for i in range(B)]
    steps = 4
    ids, cnt = syn.make_overrides(23, steps, B, D, m.vocab)
    cnt = cnt.clone()
    cnt[1] = D                                       # the step after a full commit has B * 2D rows
    max_len = max(len(p) for p in prompts) + steps * D + D
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=B, max_seq_len=max_len, D=D, tau=0.5)
    assert ctx.kernel_info == "mfma-bf16"
    st, _ = lockstep(ctx, om, prompts, D, 0.5, steps, logit_tol=2e-2, conf_tol=1e-3, overrides=(ids, cnt), bf16=True, max_len=max_len)
    assert st.step_rows[2] == B * 2 * D
    print("few rows", (B, D, hidden, ffn), st)
    ctx.close()


@pytest.mark.parametrize("lens,hidden,ffn,heads,down,gate_up", [
    ([5, 7], 3584, 6208, 2, (32, 128), (32, 64)), ([16], 2048, 6208, 2, (32, 128), (32, 64)), ([6, 8], 128, 16448, 2, (16, 32), (32, 64)),
    ([4], 64, 4608, 2, (16, 32), (16, 32)), ([1], 192, 640, 3, (16, 32), (16, 32)), ([9], 1088, 8256, 10, (16, 32), (16, 32))])
def test_bf16_few_rows_on_the_kernels_for_more(lens, hidden, ffn, heads, down, gate_up):
    """Prompts of at most 16 tokens in all: passes with separate norms, whose down projection (long k) or gate/up keeps the kernel for more rows (uneven rounds of the
    units, more than 12 rows, 32-feature blocks of one round and of more than two) or takes the streams for few.  The cached keys and values of the second and third
    layer have gone through them."""
    from paper_2509_24007_amd import sdlm
    m = mfma_cfg(n_layers=3, n_q_heads=heads, n_kv_heads=1, hidden=hidden, ffn=ffn, vocab=300, has_qkv_bias=True)
    R = sum(lens)
    assert sdlm.gemm_plan(1, R, R, hidden, ffn)[:2] == down and sdlm.gemm_plan(2, R, R, ffn, hidden)[:2] == gate_up
    om, g_dev, layers_dev = both_models(m, seed=120 + R, std=hidden ** -0.5)
    prompts = [syn.uniform_int(5, f"fm{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=len(lens), max_seq_len=32, D=4, tau=0.5)
    assert ctx.kernel_info == "mfma-bf16"
    # one step of 4 or 8 rows, each flip held to its own row's measured error; their number by those of an ideal bf16 pipeline
    ideal = orc.model_from_inputs(m, *make_model(m, seed=120 + R, std=hidden ** -0.5), bf16_points=True)
    _, seqs = lockstep(ctx, om, prompts, 4, 0.5, 1, logit_tol=2e-2, conf_tol=1e-3, bf16=True, max_len=32, floor_model=ideal)
    worst = 0.0
    for b, s in enumerate(seqs):
        for layer in range(3):
            k, v = ctx.read_kv(layer, b, 0, 0, lens[b])
            for pos in range(lens[b]):
                for got, ref in zip((k[pos].numpy(), v[pos].numpy()), s.read_kv(layer, pos, 0)):
                    worst = max(worst, float(np.max(np.abs(got - ref)) / np.max(np.abs(ref))))
    print("few rows, kernels for more", (lens, hidden, ffn, heads), worst)
    assert worst <= 2e-2
    ctx.close()


@pytest.mark.parametrize("B,D,hidden,heads,kv", [(9, 3, 192, 4, 2), (33, 1, 128, 6, 2), (11, 6, 1088, 4, 1), (17, 6, 448, 14, 2), (25, 4, 2048, 12, 2), (25, 4, 2112, 12, 2), (9, 4, 64, 28, 4),
                                                  (15, 8, 1600, 16, 2), (13, 9, 1600, 16, 2), (20, 8, 1600, 16, 2)])
def test_bf16_qkv_row_blocks(B, D, hidden, heads, kv):
    """The fused QKV launch by row blocks of 32 and of 64 and the separate kernels on the other side of its rules: ragged last
    blocks, blocks that only exist after a full commit (B * 2D rows) and are empty after single tokens, such blocks of 64 rows and of 32
    (h = 1600: 240 and 234 possible rows beside 135 and 130 certain ones, 320 beside 180; h = 2112 takes the separate kernels)."""
    m = mfma_cfg(n_layers=2, n_q_heads=heads, n_kv_heads=kv, hidden=hidden, ffn=192, vocab=1000, has_qkv_bias=True)
    om, g_dev, layers_dev = both_models(m, seed=110 + B + heads, std=0.03)
    prompts = [syn.uniform_int(5, f"rb{i}", 3 + 5 * (i % 7), 0, m.vocab - 1).numpy() for i in range(B)]
    steps = 5
    ids, cnt = syn.make_overrides(24, steps, B, D, m.vocab)
    cnt = cnt.clone()
    cnt[1] = D                                       # a step of B * 2D rows, and later one of B * (D + 1)
    cnt[3] = 1
    max_len = max(len(p) for p in prompts) + steps * D + D
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=B, max_seq_len=max_len, D=D, tau=0.5)
    assert ctx.kernel_info == "mfma-bf16"
    # gammas of eight positions flip with the roundings (20 sequences, D = 8: 12 of 100): bounded by 1.5 times (and two more than) those of an ideal bf16 pipeline as well
    ideal = orc.model_from_inputs(m, *make_model(m, seed=110 + B + heads, std=0.03), bf16_points=True)
    st, _ = lockstep(ctx, om, prompts, D, 0.5, steps, logit_tol=2e-2, conf_tol=1e-3, overrides=(ids, cnt), bf16=True, max_len=max_len, floor_model=ideal)
    assert st.step_rows[2] == B * 2 * D and st.step_rows[4] == B * (D + 1)
    print("qkv row blocks", (B, D, hidden, heads, kv), st)
    ctx.close()


@pytest.mark.parametrize("B,D,hidden,ffn,heads", [(1, 1, 64, 64, 1), (1, 8, 192, 320, 3), (8, 1, 1024, 2112, 8), (2, 4, 3072, 128, 2), (2, 4, 3136, 128, 2),
                                                   (1, 1, 3584, 64, 2), (1, 5, 4096, 64, 2), (1, 4, 4160, 448, 2), (1, 3, 8192, 64, 1), (1, 2, 8256, 64, 1)])
def test_bf16_norms_inside_the_products(B, D, hidden, ffn, heads):
    """Steps of at most 16 rows: O leaves the sums of squares and the operand of gate/up, down does so for QKV (above h = 3072 up to 4096, with the embeddings first) or
    leaves k splits to an RMSNorm; fewer k steps than wavefronts, one and 16 rows, the widest stream (8192) and one beyond it.  Three layers: first, middle, last."""
    m = mfma_cfg(n_layers=3, n_q_heads=heads, n_kv_heads=1, hidden=hidden, ffn=ffn, vocab=300, has_qkv_bias=True)
    om, g_dev, layers_dev = both_models(m, seed=160 + B, std=1.0 / hidden ** 0.5)
    prompts = [syn.uniform_int(6, f"np{i}", 3 + 4 * (i % 5), 0, m.vocab - 1).numpy() for i in range(B)]
    steps = 3
    ids, cnt = syn.make_overrides(27, steps, B, D, m.vocab)
    cnt = cnt.clone()
    cnt[1] = D                                       # then a step of B * 2D rows
    max_len = max(len(p) for p in prompts) + steps * D + D
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=B, max_seq_len=max_len, D=D, tau=0.5)
    assert ctx.kernel_info == "mfma-bf16"
    # flips of ids and gammas: at most 1.5 times (and two more than) those of an ideal bf16 pipeline on the same rows
    ideal = orc.model_from_inputs(m, *make_model(m, seed=160 + B, std=1.0 / hidden ** 0.5), bf16_points=True)
    st, _ = lockstep(ctx, om, prompts, D, 0.5, steps, logit_tol=2e-2, conf_tol=1e-3, overrides=(ids, cnt), bf16=True, max_len=max_len, floor_model=ideal)
    assert st.step_rows[2] == B * 2 * D
    print("norms inside", (B, D, hidden, ffn, heads), st)
    ctx.close()


@pytest.mark.parametrize("B,D,hidden,ffn,heads", [(17, 1, 64, 64, 2), (32, 1, 192, 16448, 6), (4, 8, 320, 448, 28), (30, 2, 2112, 192, 3), (50, 4, 128, 8256, 2),
                                                   (9, 4, 128, 640, 2), (4, 3, 2112, 8256, 2)])
def test_bf16_projections_on_the_128_row_tiles(B, D, hidden, ffn, heads):
    """Steps of 33 and more rows: projections on 128-row tiles of 128 and 256 columns, from one slice of k (no split) over divisions that leave the last
    split short to sixteen splits; gate/up of 33 to 64 rows on the 128-row tile (a matrix of more than 16384 features) and in halves with more than
    40 certain rows; 24 rows with few slices a split."""
    m = mfma_cfg(n_layers=1, n_q_heads=heads, n_kv_heads=1, hidden=hidden, ffn=ffn, vocab=300, has_qkv_bias=True)
    om, g_dev, layers_dev = both_models(m, seed=140 + B, std=0.03)
    prompts = [syn.uniform_int(5, f"pt{i}", 3 + 4 * (i % 5), 0, m.vocab - 1).numpy() for i in range(B)]
    steps = 3
    ids, cnt = syn.make_overrides(26, steps, B, D, m.vocab)
    cnt = cnt.clone()
    cnt[1] = D                                       # then a step of B * 2D rows
    max_len = max(len(p) for p in prompts) + steps * D + D
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=B, max_seq_len=max_len, D=D, tau=0.5)
    assert ctx.kernel_info == "mfma-bf16"
    st, _ = lockstep(ctx, om, prompts, D, 0.5, steps, logit_tol=2e-2, conf_tol=1e-3, overrides=(ids, cnt), bf16=True, max_len=max_len)
    assert st.step_rows[2] == B * 2 * D
    print("128-row tiles", (B, D, hidden, ffn, heads), st)
    ctx.close()


@pytest.mark.parametrize("B,D,hidden,ffn", [(5, 4, 128, 2112), (8, 4, 1408, 1088), (13, 4, 384, 2112), (16, 4, 1024, 192), (26, 4, 256, 24640), (32, 4, 128, 24576),
                                             (48, 2, 256, 24576), (48, 2, 192, 24640), (26, 4, 320, 24576)])
def test_bf16_gate_up_of_33_to_256_rows(B, D, hidden, ffn):
    """The gate/up shapes between the small-step kernel and the 128-row tiles: k in two halves inside a workgroup (one slice,
    an odd number and many slices per half; up to 64 and up to 128 rows, a ragged last column block), the 256-row tile (more
    than 128 certain rows, wide matrix; the step after a full commit has B * 2D rows, the one after single tokens B * (D + 1)) and the 192-row
    one (at most 192 possible rows, or an odd number of slices; even and odd slices, a second row block after the full commit)."""
    m = mfma_cfg(n_layers=1, n_q_heads=4, n_kv_heads=2, hidden=hidden, ffn=ffn, vocab=1000, has_qkv_bias=True)
    om, g_dev, layers_dev = both_models(m, seed=80 + B, std=0.03)
    lens = [3 + 5 * (i % 6) for i in range(B)]
    prompts = [syn.uniform_int(6, f"gu{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    steps = 5
    ids, cnt = syn.make_overrides(22, steps, B, D, m.vocab)
    cnt = cnt.clone()
    cnt[1] = D
    cnt[3] = 1
    max_len = max(lens) + steps * D + D
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=B, max_seq_len=max_len, D=D, tau=0.5)
    st, _ = lockstep(ctx, om, prompts, D, 0.5, steps, logit_tol=2e-2, conf_tol=1e-3, overrides=(ids, cnt), bf16=True, max_len=max_len)
    assert st.step_rows[2] == B * 2 * D and st.step_rows[4] == B * (D + 1)
    print("gate/up 33..256 rows", (B, D, hidden, ffn), st)
    ctx.close()


@pytest.mark.parametrize("B,D,vocab", [(1, 1, 33), (1, 4, 1001), (3, 5, 257), (9, 7, 999), (11, 16, 2050)])
def test_bf16_requested_logits_rows_and_ragged_vocabulary(B, D, vocab):
    """Requested logits leave the LM head as whole rows: every row-tile height, row counts beside a multiple of 32, vocabularies
    that end inside a wavefront's 64 entries, and nothing written outside the caller's [B * D, V]."""
    m = mfma_cfg(n_layers=1, hidden=128, ffn=192, vocab=vocab)
    om, g_dev, layers_dev = both_models(m, seed=90 + B, std=0.05)
    prompts = [syn.uniform_int(7, f"lg{i}", 2 + i, 0, vocab - 1).numpy() for i in range(B)]
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=B, max_seq_len=64, D=D, tau=0.5)
    lockstep(ctx, om, prompts, D, 0.5, 1, logit_tol=2e-2, conf_tol=1e-3, bf16=True, max_len=64)
    guard = torch.full((B * D + 2, vocab), -7.0, device="cuda")
    ids = torch.empty(B, D, dtype=torch.int32, device="cuda")
    cnt = torch.empty(B, dtype=torch.int32, device="cuda")
    ctx.decode_step(ids, cnt, None, guard[1:-1])
    torch.cuda.synchronize()
    assert (guard[0] == -7.0).all() and (guard[-1] == -7.0).all() and (guard[1:-1] != -7.0).all()
    ctx.close()


@pytest.mark.parametrize("capacity", [32, 18000])
@pytest.mark.parametrize("prompt", [100, 300, 500, 640, 980, 1500, 2100])
def test_bf16_split_kv_merge_by_number_of_chunks(prompt, capacity):
    """The split-KV merge of one sequence with 2 .. 34 chunks of 64 keys, where the context holds little more (variants by the chunks it has and may
    have), and of 1 .. 8 chunks of 512 keys where it holds far more: logits against the oracle."""
    m = mfma_cfg(n_layers=1, n_q_heads=4, n_kv_heads=2, hidden=128, ffn=192, vocab=1000)
    om, g_dev, layers_dev = both_models(m, seed=95, std=0.08)
    p = syn.uniform_int(8, f"mg{prompt}", prompt, 0, m.vocab - 1).numpy()
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=1, max_seq_len=prompt + capacity, D=4, tau=0.5)
    # flips: each one is bounded by its row's own measured logit error inside lockstep; a share of 8 rows has no meaning (random
    # logits: the top-2 gap is below twice a 6e-3 error in one row out of ten, so 2 of 8 occurs in one prompt out of five)
    lockstep(ctx, om, [p], 4, 0.5, 2, logit_tol=2e-2, conf_tol=1e-3, bf16=True, max_len=prompt + 32, flip_ceiling=1.0)
    ctx.close()


def test_bf16_split_kv_merge_of_many_groups_and_chunks():
    """Seventeen chunks of a sequence in a batch whose merge is the one for many row groups, against the same sequence alone (33 chunks, the
    merge for few groups): one step each, eager and replayed from a graph (whose launches must serve every length)."""
    m = mfma_cfg(n_layers=1, n_q_heads=8, n_kv_heads=4, hidden=128, ffn=192, vocab=1000)
    _, g_dev, layers_dev = both_models(m, seed=96, std=0.08)
    prompts = [syn.uniform_int(8, f"mm{i}", 4200 if i == 11 else 3 + i, 0, m.vocab - 1).numpy() for i in range(17)]
    out = []
    for ps, at in ((prompts, 11), ([prompts[11]], 0)):
        ctx = gpu_context(m, g_dev, layers_dev, max_batch=len(ps), max_seq_len=4300, D=4, tau=0.5, paged=True, n_pages=320, stream=torch.cuda.Stream())
        ids = torch.empty(len(ps), 4, dtype=torch.int32, device="cuda")
        cnt = torch.empty(len(ps), dtype=torch.int32, device="cuda")
        logits = torch.empty(len(ps), 4, m.vocab, device="cuda")
        for graph in (False, True):
            ctx.prefill(ps)
            ctx.graph(graph)
            ctx.decode_step(ids, cnt, None, logits)
            torch.cuda.synchronize()
            out.append(logits[at].clone())
        ctx.close()
    # two correct bf16 paths of one layer: 4 * 2^-9 of the largest logit covers the rounding of the attention output (2^-9) on its way through
    # the O projection, the MLP and the head
    for z in out[1:]:
        assert (z - out[0]).abs().max() <= 4 * 2.0 ** -9 * out[0].abs().max()


@pytest.mark.parametrize("hidden", [4100, 8200, 16384])
def test_fp32_wide_hidden_rows(hidden):
    """Rows wider than 4096 elements: the RMSNorm variants of few rows that hold two and four vectors of a row per thread (and
    the widest row the library accepts)."""
    m = gpu_cfg(hidden=hidden, n_layers=1, ffn=48, vocab=97)
    om, g_dev, layers_dev = both_models(m, seed=33, std=0.02)
    prompts = [np.array([3, 1, 4, 1, 5], dtype=np.int32), np.array([9, 2], dtype=np.int32)]
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=2, max_seq_len=32, D=3, tau=0.5)
    st, _ = lockstep(ctx, om, prompts, 3, 0.5, 3, logit_tol=1e-4, conf_tol=1e-5)
    print("wide rows", hidden, st)
    ctx.close()


@pytest.mark.parametrize("hidden,rows", [(1028, 1024), (1028, 1025), (2052, 512), (2052, 513), (4100, 256), (4100, 257), (8200, 257), (16384, 300)])
def test_fp32_rmsnorm_of_many_rows(hidden, rows):
    """Prefill passes on both sides of the rows up to which RMSNorm takes wide workgroups, and the variants of 256 threads that hold 2, 4, 8 and 16
    vectors of a row per thread: one step's logits depend on every key and value of the pass."""
    m = gpu_cfg(hidden=hidden, n_q_heads=1, n_kv_heads=1, n_layers=1, ffn=8, vocab=97)
    om, g_dev, layers_dev = both_models(m, seed=34, std=0.02)
    prompts = [syn.uniform_int(34, "rn", rows, 0, m.vocab - 1).numpy()]
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=1, max_seq_len=rows + 8, D=2, tau=0.5)
    st, _ = lockstep(ctx, om, prompts, 2, 0.5, 1, logit_tol=1e-4, conf_tol=1e-5, max_len=rows + 8)
    print("rmsnorm of many rows", hidden, rows, st)
    ctx.close()


@pytest.mark.parametrize("B,D,hidden", [(65, 3, 4160), (43, 6, 2112), (65, 7, 2112)])
def test_bf16_rmsnorm_of_many_rows_with_slabs(B, D, hidden):
    """Steps of more rows than RMSNorm takes wide workgroups for, after split-k projections (their slabs are added in the same kernel), and a step
    (43 x 6) whose certain rows are below that line and whose possible ones are above it."""
    m = mfma_cfg(n_layers=2, n_q_heads=2, n_kv_heads=1, hidden=hidden, ffn=1024, vocab=300, has_qkv_bias=True)
    # std = 1 / sqrt(h): a projection keeps the size of its input, scores have a standard deviation of sqrt(128) = 11, and the roundings of q
    # and k to bf16 (2^-9 of the value each) move them by 0.03.  At std = 0.03 (scores of 42, moved by 0.12) single attention weights are off by
    # a tenth and a logit by 3e-2, with any order of the sums.
    om, g_dev, layers_dev = both_models(m, seed=130 + B, std=hidden ** -0.5)
    prompts = [syn.uniform_int(5, f"rs{i}", 2 + i % 5, 0, m.vocab - 1).numpy() for i in range(B)]
    ids, cnt = syn.make_overrides(26, 3, B, D, m.vocab)
    cnt = cnt.clone()
    cnt[1] = D
    max_len = 8 + 4 * D
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=B, max_seq_len=max_len, D=D, tau=0.5)
    assert ctx.kernel_info == "mfma-bf16"
    st, _ = lockstep(ctx, om, prompts, D, 0.5, 3, logit_tol=2e-2, conf_tol=1e-3, overrides=(ids, cnt), bf16=True, max_len=max_len, oracle_seqs=[0, 1, B // 2, B - 1])
    print("rmsnorm with slabs", (B, D, hidden), st)
    ctx.close()


@pytest.mark.parametrize("dtype,hidden,ffn,vocab,B,D,d", [("fp32", 36, 42, 33003, 1, 5, 32), ("fp32", 68, 260, 97, 3, 3, 96), ("fp32", 260, 64, 33001, 9, 4, 128),
                                                          ("bf16", 72, 136, 33003, 3, 4, 64), ("bf16", 36, 44, 101, 2, 9, 32)])
def test_generic_row_gemm_edges(dtype, hidden, ffn, vocab, B, D, d):
    """The generic products on both sides of their dispatch: rows of whole 16-byte groups (k extents shorter than one round of
    sixteen lanes, and not a multiple of it) or not; row counts around multiples of 8 and 32; vocabularies on both sides of the
    32-row variant, ragged against its column blocks; attention lists of 1 to 6 tiles with one or two staging tiles."""
    m = gpu_cfg(hidden=hidden, ffn=ffn, vocab=vocab, n_layers=2, head_dim=d, dtype=dtype, has_qkv_bias=True)
    om, g_dev, layers_dev = both_models(m, seed=61 + B, std=0.3 if dtype == "fp32" else 0.05)
    prompts = [syn.uniform_int(6, f"rg{i}", 1 + 11 * i, 0, m.vocab - 1).numpy() for i in range(B)]
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=B, max_seq_len=160, D=D, tau=0.5, prefill_rows=33)
    bf = dtype == "bf16"
    assert ctx.kernel_info.startswith("generic")
    st, _ = lockstep(ctx, om, prompts, D, 0.5, 3, logit_tol=2e-2 if bf else 1e-4, conf_tol=1e-3 if bf else 1e-5, bf16=bf, max_len=160, verify_rule=0)
    print("generic edges", (dtype, hidden, ffn, vocab, B, D, d), st)
    ctx.close()


@pytest.mark.parametrize("dtype,d,D,paged", [("fp32", 32, 4, True), ("fp32", 96, 5, False), ("bf16", 64, 4, False), ("bf16", 32, 5, True)])
def test_generic_attention_ignores_unseen_slots(dtype, d, D, paged):
    """Cache and staging slots that a row does not see have no part in its result, whatever an earlier prompt left there: prompts of a
    token whose embedding is not a number fill pages and staging tiles (a step and its verification pass), then clean prompts use them."""
    m = gpu_cfg(head_dim=d, dtype=dtype)
    om, g_dev, layers_dev = both_models(m, seed=71, std=0.3 if dtype == "fp32" else 0.05)
    bad = m.vocab - 2
    g_dev = dict(g_dev, embed=g_dev["embed"].clone())
    g_dev["embed"][bad] = float("nan")
    lens = [1, 17, 33]
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=3, max_seq_len=96, D=D, tau=0.5, paged=paged, n_pages=18 if paged else 0)
    assert ctx.kernel_info.startswith("generic")
    ids = torch.empty(3, D, dtype=torch.int32, device="cuda")
    cnt = torch.empty(3, dtype=torch.int32, device="cuda")
    logits = torch.empty(3, D, m.vocab, device="cuda")
    ctx.prefill([[bad] * 64] * 3)
    ctx.decode_step(ids, cnt, None, logits)
    ctx.verify_step(0)
    torch.cuda.synchronize()
    assert logits.isnan().all()
    prompts = [syn.uniform_int(31, f"un{i}", n, 0, m.vocab - 3).numpy() for i, n in enumerate(lens)]
    bf = dtype == "bf16"
    _, seqs = lockstep(ctx, om, prompts, D, 0.5, 3, logit_tol=2e-2 if bf else 1e-4, conf_tol=1e-3 if bf else 1e-5, bf16=bf, max_len=96, verify_rule=0)
    assert all(bad not in [int(t) for t in s.tokens] for s in seqs)   # else the step above was not clean
    ctx.close()


@pytest.mark.parametrize("dtype,d,lead,tail", [("fp32", 32, 64, 70), ("fp32", 128, 256, 20), ("bf16", 64, 192, 3), ("bf16", 96, 320, 1)])
def test_generic_attention_keeps_non_finite_scores(dtype, d, lead, tail):
    """A score that is not a number makes the result of its row not a number, also where a wavefront has no other key in its tiles
    (runs of whole 64-key groups, of one wavefront and of all four, before the finite keys) and the values are finite.  The keys of
    one token overflow: only its embedding has feature 0, which every key weight multiplies by 3e38 or -3e38."""
    m = gpu_cfg(head_dim=d, dtype=dtype, n_layers=1, has_qkv_bias=False)
    _, g_dev, layers_dev = both_models(m, seed=72, std=0.3 if dtype == "fp32" else 0.05)
    bad = m.vocab - 2
    embed, L = g_dev["embed"].clone(), {k: v if v is None else v.clone() for k, v in layers_dev[0].items()}
    embed[:, 0] = 0
    embed[bad] = 0
    embed[bad, 0] = 1
    L["wq"][:, 0] = 0
    L["wk"][:, 0] = torch.where(torch.arange(L["wk"].shape[0], device="cuda") % 3 == 0, 3e38, -3e38).to(L["wk"].dtype)
    clean = [int(t) for t in syn.uniform_int(32, "nf", tail, 0, m.vocab - 3)]
    ctx = gpu_context(m, dict(g_dev, embed=embed), [L], max_batch=2, max_seq_len=lead + tail + 8, D=4, tau=0.5)
    assert ctx.kernel_info.startswith("generic")
    ids = torch.empty(2, 4, dtype=torch.int32, device="cuda")
    cnt = torch.empty(2, dtype=torch.int32, device="cuda")
    logits = torch.empty(2, 4, m.vocab, device="cuda")
    ctx.prefill([[bad] * lead + clean, clean])
    ctx.decode_step(ids, cnt, None, logits)
    torch.cuda.synchronize()
    k, v = ctx.read_kv(0, 0, 0, 0, lead)
    assert not k.isfinite().any() and v.isfinite().all()
    assert logits[0].isnan().all() and logits[1].isfinite().all()
    ctx.close()


@pytest.mark.parametrize("dtype,hidden,heads,kv,d,ffn,vocab,lens,D", [
    ("fp32", 264, 12, 2, 64, 1096, 97, [800], 2), ("bf16", 264, 12, 2, 64, 1096, 97, [501, 300], 2),          # QKV and gate/up by tiles, O and down by rows
    ("fp32", 260, 2, 1, 32, 72, 97, [901], 3), ("bf16", 264, 2, 1, 32, 72, 97, [450, 453], 3),                # O and down by tiles, QKV and gate/up by rows
    ("fp32", 512, 12, 2, 64, 40, 97, [1100], 1), ("fp32", 1032, 8, 2, 64, 40, 97, [1087], 1),                 # QKV, O by 32-row groups of four columns
    ("fp32", 264, 2, 1, 32, 72, 33003, [3] * 8, 4), ("bf16", 264, 2, 1, 32, 72, 33003, [3] * 9, 5),           # LM head by tiles
    ("fp32", 264, 2, 1, 32, 72, 33003, [3] * 4, 4), ("bf16", 264, 2, 1, 32, 72, 33003, [3] * 6, 4)])          # ... and just not
def test_generic_products_of_many_rows(dtype, hidden, heads, kv, d, ffn, vocab, lens, D):
    """The generic products on both sides of the line between rows without LDS and tiles, every epilogue, with ragged last rows and
    columns: prefill passes of 800 to 1100 rows (one step's logits depend on all of their keys and values) and LM heads of 16 to 45 rows."""
    m = gpu_cfg(hidden=hidden, n_q_heads=heads, n_kv_heads=kv, head_dim=d, ffn=ffn, vocab=vocab, n_layers=2 if sum(lens) < 1000 else 1, dtype=dtype)
    om, g_dev, layers_dev = both_models(m, seed=73, std=0.05)
    prompts = [syn.uniform_int(33, f"mr{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=len(lens), max_seq_len=max(lens) + 2 * D, D=D, tau=0.5)
    bf = dtype == "bf16"
    assert ctx.kernel_info.startswith("generic")
    st, _ = lockstep(ctx, om, prompts, D, 0.5, 1, logit_tol=2e-2 if bf else 1e-4, conf_tol=1e-3 if bf else 1e-5, bf16=bf, max_len=max(lens) + 2 * D)
    print("many rows", (dtype, hidden, heads, ffn, vocab, len(lens), D), st)
    ctx.close()


# ------------------------------------------------------------------ seeded random shapes
def _random_case(seed):
    rng = np.random.RandomState(seed)
    G = int(rng.choice([1, 2, 3, 4, 7, 8]))
    Hk = int(rng.choice([1, 2, 3]))
    hidden = int(rng.choice([128, 192, 256, 320, 448]))
    ffn = int(rng.choice([192, 320, 576, 1088]))
    vocab = int(rng.choice([515, 1000, 2048, 3001]))
    D = int(rng.choice([1, 2, 3, 4, 5, 8]))
    B = int(rng.choice([1, 3, 9, 17, 30]))
    lens = [int(v) for v in rng.randint(1, 70, size=B)]
    paged = bool(rng.randint(0, 2))
    kw = dict(n_q_heads=G * Hk, n_kv_heads=Hk, hidden=hidden, ffn=ffn, vocab=vocab, has_qkv_bias=bool(rng.randint(0, 2)),
              block_causal=bool(rng.randint(0, 4) == 0))
    return kw, lens, D, paged


@pytest.mark.parametrize("seed", list(range(24)))
def test_bf16_mfma_random_shapes(seed):
    """Seeded random model shapes, batch sizes, block sizes and layouts through the matrix-core path: every tile
    policy branch (row-tile height, column-tile width, split counts, ragged and possibly-empty row blocks) sees shapes
    it was not tuned on."""
    kw, lens, D, paged = _random_case(seed)
    m = mfma_cfg(**kw)
    om, g_dev, layers_dev = both_models(m, seed=100 + seed, std=0.05)
    prompts = [syn.uniform_int(seed, f"rs{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    steps = 4
    ovr = syn.make_overrides(200 + seed, steps, len(lens), D, m.vocab)
    max_len = max(lens) + steps * D + D
    n_pages = sum((n + steps * D + 15) // 16 + 1 for n in lens)
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=len(lens), max_seq_len=max_len, D=D, tau=0.5, paged=paged, n_pages=n_pages,
                      prefill_rows=int(np.random.RandomState(seed).choice([32, 64, 200])))
    assert ctx.kernel_info == "mfma-bf16"
    verify = 0 if (D >= 2 and seed % 2 == 0) else None
    st, _ = lockstep(ctx, om, prompts, D, 0.5, steps, logit_tol=2e-2, conf_tol=1e-3, overrides=ovr, bf16=True, max_len=max_len,
                     verify_rule=verify)
    print(f"random shape {seed}: {kw} B={len(lens)} D={D} paged={paged} verify={verify}", st)
    ctx.close()


@pytest.mark.parametrize("seed", list(range(12)))
def test_fp32_generic_random_shapes(seed):
    """The same for the generic kernels (fp32 debug mode): head sizes 32..128, sizes that are not multiples of any
    tile, exact ids and gamma."""
    rng = np.random.RandomState(1000 + seed)
    Hk = int(rng.choice([1, 2, 3]))
    G = int(rng.choice([1, 2, 4, 5]))
    d = int(rng.choice([32, 64, 96, 128]))
    m = gpu_cfg(n_q_heads=G * Hk, n_kv_heads=Hk, head_dim=d, hidden=int(rng.choice([36, 64, 100, 132])),
                ffn=int(rng.choice([40, 112, 250])), vocab=int(rng.choice([97, 300, 1001])),
                has_qkv_bias=bool(rng.randint(0, 2)), block_causal=bool(rng.randint(0, 4) == 0))
    D = int(rng.choice([1, 2, 3, 4, 6, 9]))
    B = int(rng.choice([1, 2, 5, 11]))
    lens = [int(v) for v in rng.randint(1, 50, size=B)]
    paged = bool(rng.randint(0, 2))
    om, g_dev, layers_dev = both_models(m, seed=300 + seed, std=0.3)
    prompts = [syn.uniform_int(seed, f"rf{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    steps = 4
    ovr = syn.make_overrides(400 + seed, steps, B, D, m.vocab)
    max_len = max(lens) + steps * D + D
    n_pages = sum((n + steps * D + 15) // 16 + 1 for n in lens)
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=B, max_seq_len=max_len, D=D, tau=0.5, paged=paged, n_pages=n_pages,
                      prefill_rows=int(rng.choice([16, 64, 200])))
    verify = int(rng.randint(0, 2)) if D >= 2 and seed % 2 == 0 else None
    st, _ = lockstep(ctx, om, prompts, D, 0.5, steps, logit_tol=1e-4, conf_tol=1e-5, overrides=ovr, max_len=max_len, verify_rule=verify)
    print(f"random fp32 shape {seed}: B={B} D={D} d={d} paged={paged} verify={verify}", st)
    assert st.id_near_tie == 0
    ctx.close()


@pytest.mark.parametrize("seed", list(range(6)))
def test_bf16_mfma_random_long_contexts(seed):
    """Few sequences with contexts of a few hundred tokens: the KV chunking policy (chunk size halves until there are
    enough work items) and the merge of many chunks see lengths on both sides of every chunk boundary."""
    rng = np.random.RandomState(2000 + seed)
    G = int(rng.choice([1, 4, 7, 16]))
    m = mfma_cfg(n_q_heads=G * 2, n_kv_heads=2, hidden=int(rng.choice([128, 256])), ffn=256, vocab=1000)
    D = int(rng.choice([2, 4, 8]))
    B = int(rng.choice([1, 2, 3]))
    lens = [int(v) for v in rng.randint(100, 520, size=B)]
    om, g_dev, layers_dev = both_models(m, seed=500 + seed, std=0.05)
    prompts = [syn.uniform_int(seed, f"rl{i}", n, 0, m.vocab - 1).numpy() for i, n in enumerate(lens)]
    steps = 3
    max_len = max(lens) + steps * D + D
    paged = bool(rng.randint(0, 2))
    n_pages = sum((n + steps * D + 15) // 16 + 1 for n in lens)
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=B, max_seq_len=max_len, D=D, tau=0.5, paged=paged, n_pages=n_pages, prefill_rows=128)
    st, _ = lockstep(ctx, om, prompts, D, 0.5, steps, logit_tol=2e-2, conf_tol=1e-3, bf16=True, max_len=max_len)
    print(f"random long {seed}: G={G} B={B} D={D} lens={lens} paged={paged}", st)
    ctx.close()


@pytest.mark.parametrize("dtype,hidden,heads,kv,d,ffn,vocab,B,D", [
    ("fp32", 64, 4, 2, 32, 112, 300, 1, 1), ("fp32", 260, 3, 1, 96, 1100, 4096, 1, 4), ("fp32", 1028, 4, 4, 64, 772, 8192, 2, 8),
    ("fp32", 768, 6, 2, 128, 700, 8200, 3, 5), ("bf16", 72, 2, 1, 32, 136, 517, 1, 7), ("bf16", 520, 8, 2, 64, 1544, 16385, 1, 16),
    ("bf16", 1032, 5, 1, 96, 520, 999, 2, 4), ("fp32", 256, 4, 2, 64, 688, 4096, 4, 4),
    ("fp32", 64, 4, 2, 32, 112, 2048, 1, 9), ("fp32", 64, 4, 2, 32, 112, 2049, 1, 9)])
def test_generic_steps_of_few_rows(dtype, hidden, heads, kv, d, ffn, vocab, B, D):
    """Steps of at most 32 rows on the generic path run norm, rotation and K/V placement inside the products, vocabulary reduction and acceptance
    in one launch: logits against the oracle, ids, confidences and counts against what the logits say.  Row counts on both sides of eight, sixteen and 32, k
    shorter than a wavefront's request and not a multiple of it, columns and vocabularies that are no whole workgroups."""
    m = gpu_cfg(dtype=dtype, hidden=hidden, n_q_heads=heads, n_kv_heads=kv, head_dim=d, ffn=ffn, vocab=vocab, n_layers=2)
    om, g_dev, layers_dev = both_models(m, seed=31, std=2.0 / hidden ** 0.5)
    prompts = [syn.uniform_int(31, f"few{i}", 5 + 14 * i, 0, vocab - 1).numpy() for i in range(B)]
    ctx = gpu_context(m, g_dev, layers_dev, max_batch=B, max_seq_len=96, D=D, tau=0.3, paged=True, n_pages=6 * B)
    ctx.prefill(prompts)
    ideal = orc.model_from_inputs(m, *make_model(m, seed=31, std=2.0 / hidden ** 0.5), bf16_points=True)
    seqs = [(orc.Seq(om, 96), orc.Seq(ideal, 96)) for _ in prompts]
    for pair, p in zip(seqs, prompts):
        for s in pair:
            s.prefill(p)
    worst = worst_ideal = 0.0
    for t in range(3):
        ids = torch.full((B, D), -1, dtype=torch.int32, device="cuda")
        cnt = torch.full((B,), -1, dtype=torch.int32, device="cuda")
        conf = torch.full((B, D), -1.0, device="cuda")
        logits = torch.full((B * D, vocab), float("nan"), device="cuda")
        ctx.decode_step(ids, cnt, conf, logits)
        p = torch.softmax(logits.double(), -1).max(-1)
        assert torch.equal(ids.view(-1).long(), logits.argmax(-1)) and (conf.view(-1) - p.values).abs().max() < 1e-5
        prod = conf.cumprod(1)
        assert torch.equal(cnt, ((prod >= 0.3).int() * torch.arange(1, D + 1, device="cuda", dtype=torch.int32)).amax(1).clamp(min=1).int())
        z = logits.view(B, D, vocab).cpu().numpy()
        pick = syn.uniform_int(32, f"o{t}", B * D, 0, vocab - 1).to(torch.int32).view(B, D)
        for b, (s, si) in enumerate(seqs):
            ref, low = s.step(D, 0.3)[0], si.step(D, 0.3)[0]
            worst = max(worst, float((np.abs(z[b] - ref).max(1) / np.abs(ref).max(1)).max()))
            worst_ideal = max(worst_ideal, float((np.abs(low - ref).max(1) / np.abs(ref).max(1)).max()))
            assert s.commit(pick[b].numpy(), (t % D) + 1) == 0 and si.commit(pick[b].numpy(), (t % D) + 1) == 0
        ctx.kv_commit(pick.cuda(), torch.full((B,), (t % D) + 1, dtype=torch.int32, device="cuda"))
    print(dtype, hidden, B, D, worst, "ideal bf16 pipeline", worst_ideal)
    # fp32: sums over at most 1544 terms, a few times sqrt(k) eps through two layers.  bf16: no further off than 1.5 times what the roundings of an ideal bf16 pipeline
    # cost on the same rows (2e-2 and more at this std: scores are wide, so that single attention weights move)
    assert worst <= (2e-5 if dtype == "fp32" else 1.5 * worst_ideal)
    ctx.close()


@pytest.mark.parametrize("path,B,D,hidden,ffn,vocab", [
    ("mfma", 1, 4, 192, 2112, 300), ("mfma", 2, 4, 1088, 4160, 300), ("mfma", 1, 3, 3136, 192, 300), ("mfma", 5, 4, 256, 1088, 300), ("mfma", 20, 4, 256, 2112, 300),
    ("fp32", 1, 4, 256, 688, 4096), ("fp32", 2, 8, 100, 250, 97), ("bf16", 1, 5, 136, 520, 1000), ("fp32", 6, 4, 64, 112, 300)])
def test_taps_leave_the_step_as_it_is(path, B, D, hidden, ffn, vocab):
    """A tapped step gives the untapped one's results bit for bit, and what its taps hold fits together: down of the tapped activation is what the residual stream
    gains, the final norm of the last stream is what enters the LM head, O of the tapped attention output is what the stream gains before."""
    dt = "fp32" if path == "fp32" else "bf16"
    m = mfma_cfg(hidden=hidden, ffn=ffn, vocab=vocab, n_layers=3) if path == "mfma" else gpu_cfg(dtype=dt, hidden=hidden, ffn=ffn, vocab=vocab, n_layers=3, head_dim=64)
    _, g_dev, layers_dev = both_models(m, seed=44, std=1.0 / hidden ** 0.5)
    prompts = [syn.uniform_int(44, f"tp{i}", 3 + 9 * i, 0, vocab - 1).numpy() for i in range(B)]
    tdt = torch.float32 if dt == "fp32" else torch.bfloat16
    nq = m.n_q_heads * m.head_dim
    out, taps = [], {}
    for tapped in (False, True):
        ctx = gpu_context(m, g_dev, layers_dev, max_batch=B, max_seq_len=300, D=D, tau=0.5)
        assert ctx.kernel_info == ("mfma-bf16" if path == "mfma" else f"generic-{dt}")
        ctx.prefill(prompts)
        ids = torch.empty(B, D, dtype=torch.int32, device="cuda")
        cnt = torch.empty(B, dtype=torch.int32, device="cuda")
        conf = torch.empty(B, D, device="cuda")
        logits = torch.empty(B * D, vocab, device="cuda")
        ctx.decode_step(ids, cnt)
        ctx.kv_commit(torch.ones(B, D, dtype=torch.int32, device="cuda"), torch.full((B,), min(D, 2), dtype=torch.int32, device="cuda"))
        if tapped:
            for which, width, t in ((0, hidden, torch.float32), (1, nq, tdt), (2, ffn, tdt), (3, hidden, torch.float32), (6, hidden, torch.float32)):
                for l in range(3):
                    taps[which, l] = torch.full((ctx.max_rows, width), float("nan"), dtype=t, device="cuda")
                    ctx.tap(l, which, taps[which, l])
            taps[4] = torch.full((B * D, hidden), float("nan"), dtype=tdt, device="cuda")
            ctx.tap(0, 4, taps[4])
        ctx.decode_step(ids, cnt, conf, logits)
        torch.cuda.synchronize()
        out.append((ids.clone(), cnt.clone(), conf.clone(), logits.clone()))
        R = len(ctx.rows()["tok"])
        kind = ctx.rows()["kind"]
        ctx.close()
    for a, b in zip(*out):
        assert torch.equal(a, b)
    f = lambda t: t[:R].double().cpu()
    for l in range(3):
        W = {k: v.double().cpu() for k, v in layers_dev[l].items() if v is not None}
        # eps of the sums: 2 sqrt(k) 2^-24 of the largest term each; 1e-5 of the largest gain covers k = 4160
        for gain, ref in ((f(taps[3, l]) - f(taps[6, l]), f(taps[2, l]) @ W["w_down"].T), (f(taps[6, l]) - f(taps[0, l]), f(taps[1, l]) @ W["wo"].T)):
            scale = max(ref.abs().max(), f(taps[3, l]).abs().max())
            assert (gain - ref).abs().max() <= 1e-5 * scale, (l, (gain - ref).abs().max().item(), scale.item())
        if l:
            assert torch.equal(taps[0, l][:R], taps[3, l - 1][:R])
    x = f(taps[3, 2])[torch.as_tensor(np.asarray(kind)) >= 0]
    xhat = x / (x.pow(2).mean(1, keepdim=True) + m.rms_eps).sqrt() * g_dev["final_norm"].double().cpu()
    assert (xhat - taps[4].double().cpu()).abs().max() <= (1e-6 if dt == "fp32" else 2.0 ** -8) * xhat.abs().max()
