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
