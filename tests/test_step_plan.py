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


def test_step_plan_rejects_bad_arguments():
    for bad in (dict(B=0, D=4), dict(B=1, D=17), dict(B=1, D=4, longest=0), dict(B=1, D=4, longest=513), dict(B=1, D=4, head_dim=48)):
        with pytest.raises(sdlm.SdlmError):
            plan(**bad)
