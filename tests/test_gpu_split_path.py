"""GPU: the split path (chunks, partial softmax states, merge) at the edges of its launch shapes,
against the numpy oracle.  Tolerances are those of gpu_common.TOL: 1e-5 where products and sums are
in fp32, the stated bf16 / fp8 bounds elsewhere."""

import pytest

import spex_workloads as sw
from gpu_common import assert_close, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


# Pieces per row from 1 to some 40 (chunks of one page), head dims whose rows take 10 to 255 threads
# of a merge workgroup (vectors of 4 or, for a head dim not divisible by 4, single elements), so
# that a row is folded in 1, 2, 4 and 8 slices and a workgroup holds one row or many.
@pytest.mark.parametrize("heads,kv_dtype", [((6, 3, 40), "f32"), ((4, 2, 64), "f32"), ((2, 1, 255), "f32"),
                                            ((4, 2, 256), "f32"), ((2, 2, 1), "f32"), ((8, 2, 128), "bf16"),
                                            ((6, 3, 30), "bf16")])
@pytest.mark.parametrize("chunk,prompt", [(1, 600), (1, 100), (3, 33), (64, 16)])
def test_merge_of_many_and_few_pieces(heads, kv_dtype, chunk, prompt):
    wl = sw.bfs_tot(n_queries=2, prompt=prompt, step=21, width=4, keep=2, depth=2, heads=heads, kv_dtype=kv_dtype,
                    q_dtype="f32" if kv_dtype == "f32" else "bf16")
    got = run_gpu(wl, prefix_chunk_pages=chunk, suffix_chunk_pages=1, kernel_mode=2)
    assert_close(got, run_oracle(wl), kv_dtype, f"{heads} {kv_dtype} chunk {chunk} prompt {prompt}")


# Row-major pools: every type; head dims at and between the padded widths 64, 128 and 256; pages of 4
# to 64 tokens (a 16-token step spans pages, or a page several steps); 1 to 140 rows per item (one,
# two, four wavefronts per row tile, several groups of 64 rows); drafts with masks; and shapes whose
# rows are not 16-byte aligned or whose pages hold fewer than four tokens (the generic kernel).
@pytest.mark.parametrize("heads,kv_dtype,page", [
    ((4, 2, 64), "f32", 16), ((4, 1, 128), "f32", 32), ((6, 3, 36), "f32", 4), ((2, 1, 256), "f32", 8), ((2, 2, 132), "f32", 16),
    ((6, 3, 40), "bf16", 16), ((8, 2, 128), "bf16", 32), ((8, 2, 128), "bf16", 4), ((28, 4, 96), "bf16", 64), ((4, 2, 256), "bf16", 16),
    ((8, 2, 64), "bf16", 8), ((10, 2, 128), "fp8_e4m3", 32), ((8, 4, 48), "fp8_e4m3", 16), ((4, 1, 256), "fp8_e4m3", 4),
    ((4, 2, 64), "fp8_e4m3", 64), ((6, 3, 20), "bf16", 16), ((4, 2, 64), "bf16", 2), ((4, 2, 24), "fp8_e4m3", 16)])
@pytest.mark.parametrize("q_len,drafts", [(1, False), (5, False), (7, True)])
def test_row_major_pools(heads, kv_dtype, page, q_len, drafts):
    wl = sw.tot_with_drafts(n_queries=2, prompt=75, step=19, depth=2, drafts=q_len, heads=heads, kv_dtype=kv_dtype,
                            q_dtype="f32" if kv_dtype == "f32" else "bf16", token_trees=drafts)
    wl.page_size = page
    for chunk in (0, 3):
        got = run_gpu(wl, prefix_chunk_pages=chunk, suffix_chunk_pages=chunk)
        assert_close(got, run_oracle(wl), "f32" if kv_dtype == "f32" else kv_dtype, f"{heads} {kv_dtype} page {page} chunk {chunk}")


def test_row_major_many_rows():
    """32 branches of 8 rows per kv head below one prompt: 256 stacked rows, four groups of 64."""
    for kv in ("f32", "bf16"):
        wl = sw.spec_at_scale(n_queries=1, prompt=130, step=20, branches=32, heads=(16, 2, 96), kv_dtype=kv,
                              q_dtype="f32" if kv == "f32" else "bf16")
        assert_close(run_gpu(wl), run_oracle(wl), kv, kv)
