"""Host logic of the forms that a decode step takes (no GPU): what the library reports is what it launches."""
import itertools

import pytest

from helpers import small_cfg
from paper_2509_24007_amd import sdlm

SEPARATE, GENERIC, MFMA, MFMA_WHOLE = 0, 1, 2, 3
LAUNCH, ASSEMBLY, CHAIN = 0, 1, 2


def plan(B, D, **kw):
    run = {k: kw.pop(k) for k in ("committed", "longest", "max_seq_len") if k in kw}
    m = small_cfg(**dict(dict(dtype="bf16", hidden=1536, n_q_heads=12, n_kv_heads=2, head_dim=128, ffn=8960, vocab=1000), **kw))
    return sdlm.step_plan(sdlm.model_cfg(m), B, D, **run)


def test_embeddings_are_gathered_once():
    """A chain whose layers start without a norm gathers them itself, with the first operands; the row assembly then leaves them alone."""
    p = plan(1, 1, hidden=3584, n_q_heads=28, n_kv_heads=4, ffn=18944)
    assert p["chain"] == MFMA_WHOLE and p["embeds"] == CHAIN
    for h, B, D, hd in itertools.product((64, 512, 3072, 3136, 4096, 4160, 8192), (1, 2, 5), (1, 2, 4), (64, 128)):
        p = plan(B, D, hidden=h, n_q_heads=2, n_kv_heads=1, head_dim=hd)
        assert (p["embeds"] == CHAIN) == (p["chain"] == MFMA_WHOLE) == (hd == 128 and B * 2 * D <= 16 and 3072 < h <= 4096), (h, B, D, hd, p)
        if p["embeds"] != CHAIN:
            assert (p["embeds"] == ASSEMBLY) == (B <= 4 and B * 2 * D * h <= 8192)


@pytest.mark.parametrize("dtype,h,F,hq,hk,d,B,D,few", [
    # layers on both sides of the lines, eight rows and more: bf16 160, 45, 18 and 9 million weights, fp32 360, 150, 80 and 50
    ("fp32", 256, 688, 4, 2, 64, 1, 4, True), ("fp32", 256, 688, 4, 2, 64, 4, 4, True), ("fp32", 256, 688, 4, 2, 64, 5, 4, False),
    ("bf16", 896, 4864, 14, 2, 64, 1, 4, True), ("bf16", 896, 4864, 14, 2, 64, 4, 4, True), ("bf16", 896, 4864, 14, 2, 64, 16, 1, False),
    ("bf16", 1800, 9720, 9, 9, 96, 3, 4, False), ("bf16", 1800, 9720, 9, 9, 96, 1, 4, True), ("bf16", 4000, 16000, 125, 125, 32, 4, 2, False),
    ("bf16", 2856, 15416, 89, 1, 32, 4, 4, False), ("bf16", 3848, 13464, 120, 1, 32, 1, 4, False),
    ("fp32", 2048, 11008, 16, 2, 128, 4, 4, True), ("fp32", 2712, 14640, 42, 2, 64, 4, 4, False), ("fp32", 3976, 15904, 31, 31, 64, 2, 5, False),
    ("fp32", 3976, 15904, 31, 31, 64, 1, 4, True)])
def test_generic_steps_of_few_rows_by_the_size_of_a_layer(dtype, h, F, hq, hk, d, B, D, few):
    p = plan(B, D, dtype=dtype, hidden=h, ffn=F, n_q_heads=hq, n_kv_heads=hk, head_dim=d)
    assert p["chain"] == (GENERIC if few else SEPARATE) and p["attn"] == -1 and p["qkv_rows"] == 0
    # rows that are no whole 16-byte pieces never
    assert plan(B, D, dtype=dtype, hidden=h, ffn=F + 2, n_q_heads=hq, n_kv_heads=hk, head_dim=d)["chain"] == SEPARATE


@pytest.mark.parametrize("dtype,V,B,D,head", [("fp32", 4096, 1, 4, 2), ("fp32", 5000, 1, 8, 2), ("fp32", 5001, 1, 8, 1), ("fp32", 2501, 1, 9, 1), ("fp32", 1250, 8, 4, 2), ("fp32", 300, 33, 1, 1),
                                              ("bf16", 3000, 2, 4, 2), ("bf16", 4227, 2, 16, 1), ("bf16", 5106, 8, 4, 1), ("bf16", 4653, 4, 5, 1), ("bf16", 750, 2, 16, 2)])
def test_generic_head_by_columns_and_rows(dtype, V, B, D, head):
    assert plan(B, D, dtype=dtype, hidden=256, ffn=688, n_q_heads=4, n_kv_heads=2, head_dim=64, vocab=V)["lm_head"] == head


@pytest.mark.parametrize("V,D,one", [(16384, 1, 1), (16385, 1, 0), (16384, 8, 1), (2048, 9, 1), (2049, 9, 0), (16384, 16, 0), (97, 16, 1)])
def test_reduction_and_acceptance_in_one_launch_by_threads_a_row(V, D, one):
    for B in (1, 64):
        assert plan(B, D, dtype="fp32", hidden=64, ffn=64, n_q_heads=2, n_kv_heads=1, head_dim=32, vocab=V)["lm_accept"] == one
    assert plan(1, D, vocab=V)["lm_accept"] == 0


def test_step_plan_rejects_bad_arguments():
    for bad in (dict(B=0, D=4), dict(B=1, D=17), dict(B=1, D=4, longest=0), dict(B=1, D=4, longest=513), dict(B=1, D=4, head_dim=48)):
        with pytest.raises(sdlm.SdlmError):
            plan(**bad)
