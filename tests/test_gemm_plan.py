"""Host logic of the matrix-core GEMM launch policy (no GPU): invariants over a sweep of problem shapes.

The policy picks a kernel and workgroup tile (rows x columns) and a number of splits along k.  Whatever it picks must be a shape
the kernels can run correctly: the tile is one of the compiled ones, every split owns a part of k (64-deep slices in the tiled
kernel, 32-deep steps in the one for few rows; an empty split would leave its partial-sum slab unwritten), the slabs fit the scratch
area, and epilogues that need the whole sum (SiLU(gate)*up, LM head) are never split.  The library launches what it reports."""
import itertools

import pytest

from paper_2509_24007_amd import sdlm

SLAB_FLOATS = 16 << 20
STORE, RESID, SWIGLU, LMHEAD = 0, 1, 2, 3


def slices_per_split(k, splits):
    s = k // 64
    return (s + splits - 1) // splits


@pytest.mark.parametrize("epi", [STORE, RESID, SWIGLU, LMHEAD])
def test_policy_invariants(epi):
    rows_list = [1, 5, 8, 31, 32, 33, 48, 64, 65, 100, 144, 160, 192, 256, 323, 384, 512, 960, 2048, 4096]
    n_list = [128, 130, 512, 1088, 2048, 2560, 3584, 4608, 5120, 7168, 8960, 18944, 27648, 151936]
    k_list = [64, 128, 192, 1536, 2048, 2688, 3584, 5120, 8960, 18944, 27648]
    seen = set()
    for rows, n, k in itertools.product(rows_list, n_list, k_list):
        for min_rows in {0, rows, max(1, rows // 2), max(1, (rows * 5) // 8)}:
            tr, tc, sp = sdlm.gemm_plan(epi, rows, min_rows, n, k)
            seen.add((tr, tc))
            few = (tr, tc) == (16, 32) or (epi == SWIGLU and (tr, tc) == (32, 64))
            halves = epi == SWIGLU and tc == 128                               # k in halves inside the workgroup
            if few:
                # kernels without LDS tiles: they serve no rows beyond their tile
                assert epi in (RESID, SWIGLU) and rows <= tr
                if sp > 1:
                    assert epi == RESID and 1 < sp <= 16 and sp <= k // 32 and sp * rows * n <= SLAB_FLOATS, (rows, n, k, sp)
                continue
            assert tr in (32, 64, 128, 192, 256) and tc in (128, 256, 512), (rows, n, k, tr, tc)
            assert tr < 192 or (epi == SWIGLU and tc == 256)                  # the 192- and 256-row tiles exist for gate/up only
            assert tc >= 256 or epi in (STORE, RESID) or halves                # the narrow tile has only the plain epilogues
            if halves:
                # two equal halves of whole slices; one row block; compiled for 64 and 128 rows
                assert k % 128 == 0 and tr in (64, 128) and 32 < rows <= tr
            if tr == 256:
                # an even number of slices; only where more than one row block of 192 would be needed, and a certain row in it
                assert k % 128 == 0 and rows > 192 and 128 < min_rows <= 192, (rows, min_rows, n, k)
            if tr == 192:
                assert 128 < min_rows <= 192 and (rows <= 192 or k % 128)
            if tc == 512:
                # the eight-wavefront tile: 128 rows, never split, only where the four-wavefront launch would have put more
                # workgroups on the chip than it has compute units; not compiled for the plain-store and LM-head epilogues
                assert tr == 128 and sp == 1 and epi in (RESID, SWIGLU)
                col_blocks4 = -(-n // 128) if epi == SWIGLU else -(-n // 256)
                sure_row_blocks = max(1, min(-(-rows // 128), -(-min_rows // 128))) if min_rows > 0 else -(-rows // 128)
                assert col_blocks4 * sure_row_blocks > 256, (rows, min_rows, n, k)
            # up to 32 rows the tiled kernel runs O and down (and the LM head) only, on 32-row tiles: gate/up and QKV have kernels without LDS tiles there
            assert rows > 32 or tr == (128 if epi == STORE else 32)
            assert sp >= 1
            if epi in (SWIGLU, LMHEAD):
                assert sp == 1
            per = slices_per_split(k, sp)
            assert (sp - 1) * per < k // 64 <= sp * per, f"empty or missing split: rows={rows} n={n} k={k} splits={sp}"
            if sp > 1:
                assert sp * rows * n <= SLAB_FLOATS, (rows, n, k, sp)
                assert sp <= 16
    if epi == RESID:
        assert (16, 32) in seen
    if epi == SWIGLU:
        assert {(16, 32), (32, 64), (64, 128), (128, 128), (192, 256), (256, 256), (64, 256), (128, 256), (128, 512)} <= seen
    if epi in (STORE, RESID):
        assert (128, 128) in seen and (128, 256) in seen                            # the sweep reaches both widths
        assert ((32, 128) in seen) == (epi == RESID)


def test_policy_on_the_benchmark_shapes():
    # the 7B shape at 323 typical rows (capacity 512, 320 certain): one workgroup per compute unit for the long-k
    # projection, few splits for the short-k ones, the 192-row tile only for the 32B gate/up
    assert sdlm.gemm_plan(RESID, 512, 320, 3584, 18944) == (128, 256, 6)
    tr, tc, sp = sdlm.gemm_plan(RESID, 512, 320, 3584, 3584)
    assert sp <= 3
    tr, tc, sp = sdlm.gemm_plan(STORE, 512, 320, 4608, 3584)
    assert sp <= 3
    assert sdlm.gemm_plan(SWIGLU, 512, 320, 18944, 3584) == (128, 512, 1)             # 444 workgroups of four wavefronts: eight instead
    # the 32B gate/up of a step of 160 certain and up to 256 rows is one row block, whatever rows there are; up to 192 the 192-row tile
    assert sdlm.gemm_plan(SWIGLU, 256, 160, 27648, 5120) == (256, 256, 1)
    assert sdlm.gemm_plan(SWIGLU, 192, 144, 27648, 5120) == (192, 256, 1)
    assert sdlm.gemm_plan(SWIGLU, 256, 144, 11008, 2048)[0] == 128               # too few column blocks for the tall tile
    assert sdlm.gemm_plan(LMHEAD, 256, 256, 151936, 3584) == (128, 256, 1)
    # passes of few rows outside the chain of a step's own (prompts of at most 16 tokens, steps of 17 to 32 rows): streams without LDS tiles, at most 16 k splits
    assert sdlm.gemm_plan(SWIGLU, 8, 5, 8960, 1536) == (16, 32, 1) and sdlm.gemm_plan(SWIGLU, 32, 20, 8960, 1536) == (32, 64, 1)
    assert sdlm.gemm_plan(RESID, 8, 5, 1536, 8960) == (16, 32, 10) and sdlm.gemm_plan(RESID, 8, 5, 1536, 1536) == (16, 32, 3)
    # ... and where they lose, the kernels for more rows: long k with workgroups between one and two rounds of the units, 13 to 16 rows
    assert sdlm.gemm_plan(RESID, 8, 5, 3584, 18944) == (32, 128, 16) and sdlm.gemm_plan(RESID, 16, 16, 3584, 3584) == (16, 32, 4)
    assert sdlm.gemm_plan(RESID, 16, 16, 2048, 11008) == (32, 128, 16) and sdlm.gemm_plan(RESID, 16, 10, 2048, 11008) == (16, 32, 8)
    assert sdlm.gemm_plan(RESID, 16, 16, 5120, 27648) == (16, 32, 3) and sdlm.gemm_plan(RESID, 16, 16, 1536, 8960) == (16, 32, 10)
    assert sdlm.gemm_plan(SWIGLU, 16, 16, 18944, 3584) == (32, 64, 1) and sdlm.gemm_plan(SWIGLU, 16, 10, 18944, 3584) == (16, 32, 1)
    assert sdlm.gemm_plan(SWIGLU, 16, 5, 6912, 2560) == (32, 64, 1) and sdlm.gemm_plan(SWIGLU, 16, 16, 11008, 2048) == (16, 32, 1)
    # gate/up of 33 to 128 rows: k in halves where the 64-feature blocks are one round of the compute units
    assert sdlm.gemm_plan(SWIGLU, 66, 66, 11008, 2048) == (128, 128, 1) and sdlm.gemm_plan(SWIGLU, 64, 40, 8960, 1536) == (64, 128, 1)
    assert sdlm.gemm_plan(SWIGLU, 70, 42, 18944, 3584) == (128, 256, 1)
    # a 4096-row prefill pass of the 7B shape: unsplit everywhere; the residual projections and gate/up take the wide tile
    assert sdlm.gemm_plan(RESID, 4096, 4096, 3584, 18944) == (128, 512, 1)
    assert sdlm.gemm_plan(SWIGLU, 4096, 4096, 18944, 3584) == (128, 512, 1)
    assert sdlm.gemm_plan(STORE, 4096, 4096, 4608, 3584) == (128, 256, 1)


def test_projections_between_one_and_two_rounds_of_the_units():
    # measured choices where the weights begin to be shared (250 to 500 rows) and where a second workgroup on a unit costs more than it saves
    assert sdlm.gemm_plan(STORE, 630, 378, 3840, 3072) == (128, 128, 2)
    assert sdlm.gemm_plan(STORE, 410, 410, 3584, 3072) == (128, 128, 2) and sdlm.gemm_plan(STORE, 451, 451, 3072, 2560) == (128, 128, 2)
    assert sdlm.gemm_plan(RESID, 410, 410, 3072, 3072) == (128, 128, 2)
    assert sdlm.gemm_plan(RESID, 274, 274, 6144, 24576) == (128, 256, 3)
    assert sdlm.gemm_plan(RESID, 572, 572, 5120, 27136) == (128, 256, 2)


def test_plan_rejects_bad_arguments():
    with pytest.raises(sdlm.SdlmError):
        sdlm.gemm_plan(0, 0, 0, 128, 128)
    with pytest.raises(sdlm.SdlmError):
        sdlm.gemm_plan(0, 8, 0, 128, 100)
    with pytest.raises(sdlm.SdlmError):
        sdlm.gemm_plan(7, 8, 0, 128, 128)
