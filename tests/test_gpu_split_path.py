"""GPU: the split path (chunks, partial softmax states, merge) at the edges of its launch shapes,
against the numpy oracle.  Tolerances are those of gpu_common.TOL: 1e-5 where products and sums are
in fp32, the stated bf16 / fp8 bounds elsewhere."""

import math

import numpy as np
import pytest
import torch

import spex_workloads as sw
from gpu_common import assert_close, build_gpu_tree, run_gpu, run_oracle, run_oracle_c

pytestmark = pytest.mark.gpu
THROUGH_LDS, ONE_REGISTER_SET, ROW_TILES = range(3)  # SpexTree.split_form


def run_form(wl, form, **kw):
    """As run_gpu on the split path, which has to take the form named."""
    tree = build_gpu_tree(wl, kernel_mode=2, **kw)
    got = run_gpu(wl, tree=tree)
    ran = tree.split_form()
    tree.close()
    assert ran == form, f"{wl.name}: form {ran}, not {form}"
    return got


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


# Pieces' records at a fixed stride (all query tokens with the same number, or one short of it, the rest filled up) and
# through part_indptr (uneven prompts); 1, 3, 4, 8 and 16 kv heads; 2 to 24 heads each, more and fewer than the rows of a workgroup.
@pytest.mark.parametrize("heads", [(2, 1, 64), (24, 1, 128), (12, 3, 40), (20, 4, 128), (8, 8, 64), (32, 16, 64)])
@pytest.mark.parametrize("prompts", [(64, 64), (64, 64, 64, 48), (16, 300)])
def test_merge_records_at_a_stride(heads, prompts):
    import paper_2605_10195_amd as spex
    gen = torch.Generator().manual_seed(len(prompts))
    Hq, Hkv, D = heads
    kv = "bf16" if D >= 64 else "f32"
    dt = torch.bfloat16 if kv == "bf16" else torch.float32
    t = spex.SpexTree(Hq, Hkv, D, 16, kv, kv, num_pages=200, device="cuda", kernel_mode=2, prefix_chunk_pages=1, suffix_chunk_pages=1)
    leaves, paths = [], []
    for n in prompts:
        (root,) = t.fork(-1, 1)
        k, v = (torch.randn((n, Hkv, D), generator=gen).to(dt) for _ in range(2))
        t.append_step(root, k.cuda(), v.cuda())
        for u in t.fork(root, 2):
            ku, vu = (torch.randn((20, Hkv, D), generator=gen).to(dt) for _ in range(2))
            t.append_step(u, ku.cuda(), vu.cuda())
            leaves.append(u)
            paths.append((torch.cat([k, ku]).double(), torch.cat([v, vu]).double()))
    q = torch.randn((len(leaves), Hq, D), generator=gen).to(dt)
    out, lse = t.decode_attention(leaves, None, q.cuda(), D ** -0.5)
    for i, (k, v) in enumerate(paths):
        s = torch.einsum("hd,thd->ht", q[i].double(), k.repeat_interleave(Hq // Hkv, dim=1)) * D ** -0.5
        want = torch.einsum("ht,thd->hd", torch.softmax(s, dim=1), v.repeat_interleave(Hq // Hkv, dim=1))
        tol = 1e-5 if kv == "f32" else 1e-3     # gpu_common.TOL
        assert float((out[i].double().cpu() - want).norm() / want.norm()) <= tol
        assert float((lse[i].double().cpu() - torch.logsumexp(s, dim=1)).abs().max()) <= tol
    t.close()


# Merge workgroups of several query tokens (1 to 3 heads a kv head): fewer query tokens than one holds, as many, one more and many, in 1
# to 8 slices; the last case in phases, which merge a list of query tokens.
@pytest.mark.parametrize("heads,kv_dtype", [((8, 8, 64), "bf16"), ((16, 8, 128), "bf16"), ((6, 3, 40), "f32"), ((2, 2, 1), "f32"), ((3, 3, 255), "f32"),
                                            ((12, 4, 96), "fp8_e4m3")])
@pytest.mark.parametrize("queries,width,prompt,chunk", [(1, 1, 40, 1), (1, 5, 200, 1), (3, 5, 20, 0), (4, 4, 20, 0), (11, 3, 20, 0), (24, 11, 70, 2)])
def test_merge_of_several_query_tokens(heads, kv_dtype, queries, width, prompt, chunk):
    wl = sw.bfs_tot(n_queries=queries, prompt=prompt, step=21, width=width, keep=width, depth=1, heads=heads, kv_dtype=kv_dtype,
                    q_dtype="f32" if kv_dtype == "f32" else "bf16")
    got = run_gpu(wl, prefix_chunk_pages=chunk, suffix_chunk_pages=chunk, kernel_mode=2)
    assert_close(got, run_oracle_c(wl), kv_dtype, f"{heads} {kv_dtype} {queries} x {width}")


@pytest.mark.parametrize("heads", [(8, 8, 64), (16, 8, 64)])
def test_merge_list_of_several_query_tokens_a_workgroup(heads):
    wl = sw.random_trace(78, heads=heads, n_ops=1200, n_roots=250)
    got = run_gpu(wl, kernel_mode=2, prefix_chunk_pages=1, suffix_chunk_pages=3)
    assert_close(got, run_oracle_c(wl), "bf16", f"{heads}")


# Row-major pools: every type; head dims at and between the padded widths 64, 128 and 256; pages of 4
# to 64 tokens (a 16-token step spans pages, or a page several steps); 1 to 140 rows per item (one,
# two, four wavefronts per row tile, several groups of 64 rows); drafts with masks; fp8 rows of 8 and not of
# 16 bytes (heads of 24 and 40); and shapes whose rows are not 16-byte (fp8 8-byte) aligned or whose pages hold fewer
# than four tokens (the generic kernel: bf16 heads of 20, fp8 heads of 20 and 136, pages of two).
@pytest.mark.parametrize("heads,kv_dtype,page", [
    ((4, 2, 64), "f32", 16), ((4, 1, 128), "f32", 32), ((6, 3, 36), "f32", 4), ((2, 1, 256), "f32", 8), ((2, 2, 132), "f32", 16),
    ((6, 3, 40), "bf16", 16), ((8, 2, 128), "bf16", 32), ((8, 2, 128), "bf16", 4), ((28, 4, 96), "bf16", 64), ((4, 2, 256), "bf16", 16),
    ((8, 2, 64), "bf16", 8), ((10, 2, 128), "fp8_e4m3", 32), ((8, 4, 48), "fp8_e4m3", 16), ((4, 1, 256), "fp8_e4m3", 4),
    ((4, 2, 64), "fp8_e4m3", 64), ((6, 3, 20), "bf16", 16), ((4, 2, 64), "bf16", 2), ((4, 2, 24), "fp8_e4m3", 16),
    ((6, 3, 40), "fp8_e4m3", 4), ((4, 2, 20), "fp8_e4m3", 16), ((4, 2, 136), "fp8_e4m3", 16)])
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


# Row 0: every score between -8e37 and -2e37, so that the first token takes all the weight.  Row 1: scores
# that rise by less than 2^8 in weight from token to token and over all, and values whose sum under weights
# of at most 1 stays below the end of fp32.  fp32 weights and sums throughout: 1e-5 as elsewhere.
@pytest.mark.parametrize("kv", ["f32", "bf16"])
@pytest.mark.parametrize("n_tokens,chunk", [(1, 0), (7, 0), (300, 0), (300, 1)])
def test_row_major_scores_and_values_at_the_end_of_the_range(kv, n_tokens, chunk):
    import paper_2605_10195_amd as spex
    dt = torch.float32 if kv == "f32" else torch.bfloat16
    heads, dim, page = 2, 40, 16
    t = spex.SpexTree(heads, 1, dim, page, kv, kv, num_pages=-(-n_tokens // page) + 1, device="cuda", prefix_chunk_pages=chunk,
                      suffix_chunk_pages=chunk)
    (u,) = t.fork(-1, 1)
    k = torch.zeros((n_tokens, 1, dim))
    k[:, 0, 0] = 2e18 * (1.0 + 3.0 * torch.arange(n_tokens) / n_tokens)
    v = (1e36 * (0.5 + 0.5 * torch.arange(n_tokens) / n_tokens))[:, None, None].repeat(1, 1, dim)
    k, v = k.to(dt).cuda(), v.to(dt).cuda()
    t.append_step(u, k, v)
    q = torch.zeros((1, heads, dim))
    q[0, 0, 0], q[0, 1, 0] = -1e19, 5.0 / 8e18
    q = q.to(dt).cuda()
    out, lse = t.decode_attention([u], None, q, 1.0)
    s = q[0, :, :1].double().cpu() * k[:, 0, 0].double().cpu()
    want, got = torch.softmax(s, dim=1) @ v[:, 0].double().cpu(), out[0].double().cpu()
    assert bool(torch.isfinite(got).all())
    assert float((got / want - 1.0).abs().max()) <= 1e-5
    assert float((lse[0].double().cpu() / torch.logsumexp(s, dim=1) - 1.0).abs().max()) <= 1e-5
    t.close()


# 16-bit and fp8 rows: tokens go through the kernel 32 at a time, two groups of 16, split between one, two or four
# wavefronts, so counts around multiples of 16; pages that hold a step and pages of four tokens; head dims equal to a
# padded width and below it; fp8 rows of 8 and not of 16 bytes up to 128 dims, and beyond them in the generic kernel.
# Weights are fp32 and products exact: 2e-6 is four times the error of fp32 sums of this length (5e-7).  An infinite
# value reaches every row that sees its token, as +-inf and not as NaN.
@pytest.mark.parametrize("kv,dim", [("bf16", 64), ("bf16", 96), ("bf16", 128), ("bf16", 256), ("fp8_e4m3", 48), ("fp8_e4m3", 128),
                                    ("fp8_e4m3", 256), ("fp8_e4m3", 8), ("fp8_e4m3", 40), ("fp8_e4m3", 120), ("fp8_e4m3", 136)])
@pytest.mark.parametrize("n_tokens", [1, 15, 17, 32, 33, 48, 161, 300])
@pytest.mark.parametrize("heads", [2, 20])
@pytest.mark.parametrize("page", [32, 4])
def test_row_major_sums_keep_fp32_weights(kv, dim, n_tokens, heads, page):
    import paper_2605_10195_amd as spex
    gen = torch.Generator().manual_seed(n_tokens + dim)
    pages = -(-n_tokens // page)
    t = spex.SpexTree(heads, 1, dim, page, "bf16", kv, num_pages=pages, device="cuda", pool_fill=255)
    (u,) = t.fork(-1, 1)
    k, v = (torch.randn((n_tokens, 1, dim), generator=gen) for _ in range(2))
    scale = torch.ones((pages, 1))
    if kv == "bf16":
        k, v = k.to(torch.bfloat16), v.to(torch.bfloat16)
        v[n_tokens // 2, 0, 3] = float("inf")
        t.append_step(u, k.cuda(), v.cuda())
    else:
        k, v = k.to(torch.float8_e4m3fn), v.to(torch.float8_e4m3fn)
        scale = torch.rand((pages, 1), generator=gen) + 0.5
        t.append_step(u, k.view(torch.uint8).cuda(), v.view(torch.uint8).cuda(), scale.cuda(), scale.cuda())
    q = torch.randn((1, heads, dim), generator=gen).to(torch.bfloat16)
    out, lse = t.decode_attention([u], None, q.cuda(), dim ** -0.5)
    f = scale.double().repeat_interleave(page)[:n_tokens, None]
    kd, vd = k[:, 0].double() * f, v[:, 0].double() * f
    s = q[0].double() @ kd.T * dim ** -0.5
    want, got = torch.softmax(s, dim=1) @ vd, out[0].double().cpu()
    if kv == "bf16":
        assert bool((got[:, 3] == float("inf")).all())
        want[:, 3] = got[:, 3] = 0.0
    assert float((got - want).norm() / want.norm()) <= 2e-6
    assert float((lse[0].double().cpu() - torch.logsumexp(s, dim=1)).abs().max()) <= 2e-6 * (1.0 + math.log(n_tokens))
    t.close()


# Weights 2^-drop of the row's largest, which a token without a value has (one in every 16, so that every wavefront meets
# it), and fp8 page scales as small: below 2^-110 a bf16 piece no longer holds a weight's last bits.  Scores are multiples
# of 1/16 and exact in fp32, so the bound is that of the sums above.
@pytest.mark.parametrize("kv,dim", [("bf16", 40), ("bf16", 64), ("bf16", 128), ("bf16", 256), ("fp8_e4m3", 40), ("fp8_e4m3", 64),
                                    ("fp8_e4m3", 128), ("fp8_e4m3", 256)])
@pytest.mark.parametrize("drop", [20, 85, 88, 112, 118, 124])
@pytest.mark.parametrize("n_tokens", [16, 45])
def test_row_major_weights_far_below_the_largest(kv, dim, drop, n_tokens):
    import paper_2605_10195_amd as spex
    gen = torch.Generator().manual_seed(drop + dim)
    heads, page = 6, 32
    pages = -(-n_tokens // page)
    t = spex.SpexTree(heads, 1, dim, page, "bf16", kv, num_pages=pages, device="cuda", pool_fill=255)
    (u,) = t.fork(-1, 1)
    at = torch.arange(n_tokens)
    k = torch.zeros((n_tokens, 1, dim))
    k[at % 16 != 0, 0, 0] = -1.0
    k[:, 0, 1] = -(at % 16) / 16.0
    v = torch.rand((n_tokens, 1, dim), generator=gen) + 0.5
    v[at % 16 == 0] = 0.0
    q = torch.zeros((1, heads, dim))
    q[0, :, 1] = 1.0
    scale = 1.0
    if kv == "bf16":
        q[0, :, 0] = drop
        k, v = k.to(torch.bfloat16), (1e36 * v).to(torch.bfloat16)
        v[n_tokens - 1, 0, 3] = float("inf")
        t.append_step(u, k.cuda(), v.cuda())
    else:
        scale = 1.3712 * 2.0 ** -drop
        k, v = k.to(torch.float8_e4m3fn), v.to(torch.float8_e4m3fn)
        s_v = torch.full((pages, 1), scale)
        scale = s_v[0, 0].double()
        t.append_step(u, k.view(torch.uint8).cuda(), v.view(torch.uint8).cuda(), torch.ones((pages, 1)).cuda(), s_v.cuda())
    out, _ = t.decode_attention([u], None, q.to(torch.bfloat16).cuda(), math.log(2.0))
    s = q[0].double() @ k[:, 0].double().T * math.log(2.0)
    want, got = torch.softmax(s, dim=1) @ (v[:, 0].double() * scale), out[0].double().cpu()
    if kv == "bf16":
        assert bool((got[:, 3] == float("inf")).all())
        want[:, 3] = got[:, 3] = 0.0
    assert float((got - want).norm() / want.norm()) <= 2e-6
    t.close()


# Pages of 4 and 8 tokens: a group of 16 tokens may reach past an item's pages, where the kernel reads tokens of the last
# page again.  An infinite value there, visible to every row, gives +-inf; a repetition of it under weight 0 would give NaN.
@pytest.mark.parametrize("kv", ["f32", "bf16"])
@pytest.mark.parametrize("page", [4, 8, 16])
@pytest.mark.parametrize("n_tokens", [1, 4, 9, 12, 20, 24, 40, 44, 100])
@pytest.mark.parametrize("chunk", [0, 3])
def test_row_major_infinite_value_in_the_last_page(kv, page, n_tokens, chunk):
    import paper_2605_10195_amd as spex
    dt, dim = (torch.float32 if kv == "f32" else torch.bfloat16), 40
    gen = torch.Generator().manual_seed(n_tokens)
    t = spex.SpexTree(3, 1, dim, page, kv, kv, num_pages=-(-n_tokens // page), device="cuda", pool_fill=255, prefix_chunk_pages=chunk,
                      suffix_chunk_pages=chunk)
    (u,) = t.fork(-1, 1)
    k, v = (torch.randn((n_tokens, 1, dim), generator=gen).to(dt) for _ in range(2))
    v[n_tokens - 1, 0, 3] = float("inf")
    v[(n_tokens - 1) // page * page, 0, 5] = float("-inf")
    t.append_step(u, k.cuda(), v.cuda())
    q = torch.randn((1, 3, dim), generator=gen).to(dt)
    got = t.decode_attention([u], None, q.cuda(), dim ** -0.5)[0][0].double().cpu()
    assert bool((got[:, 3] == float("inf")).all()) and bool((got[:, 5] == float("-inf")).all())
    v[:, 0, 3] = v[:, 0, 5] = 0.0
    got[:, 3] = got[:, 5] = 0.0
    want = torch.softmax(q[0].double() @ k[:, 0].double().T * dim ** -0.5, dim=1) @ v[:, 0].double()
    assert float((got - want).norm() / want.norm()) <= 2e-6   # fp32 weights and sums, as above
    t.close()


@pytest.mark.parametrize("chunk", [64, 4, 1])
def test_lse_of_a_row_whose_scores_overflow(chunk):
    """All scores of head 0 are -inf in fp32: its lse is -inf however many pieces and slices the merge folds;
    head 1 is not touched by it."""
    import paper_2605_10195_amd as spex
    t = spex.SpexTree(2, 1, 40, 16, "f32", "f32", num_pages=32, device="cuda", prefix_chunk_pages=chunk, suffix_chunk_pages=chunk)
    (u,) = t.fork(-1, 1)
    k = torch.full((300, 1, 40), 1e30, device="cuda")
    t.append_step(u, k, torch.ones_like(k))
    q = torch.zeros((1, 2, 40), device="cuda")
    q[0, 0] = -1e30
    out, lse = t.decode_attention([u], None, q, 1.0)
    assert float(lse[0, 0]) == float("-inf")
    assert abs(float(lse[0, 1]) - math.log(300)) <= 1e-5 and float((out[0, 1] - 1.0).abs().max()) <= 1e-5
    t.close()


def _single_pieces(n, **kw):
    return sw.bfs_tot(n_queries=n, prompt=40, step=20, width=1, keep=1, depth=1, **kw)


# Launches of many items go in phases: with more than 16 private rows beyond 512 workgroups, else beyond 4096
# private items (head dim 64).  Either side of both bounds: draft masks on fp8, requests of 71 rows (three row
# spans), 4 rows, and requests of one piece each, which no merge follows.
@pytest.mark.parametrize("make", [
    lambda more: sw.tot_with_drafts(n_queries=8 + more, prompt=75, step=19, depth=2, drafts=6, heads=(40, 8, 128), token_trees=True),
    lambda more: sw.tot_with_drafts(n_queries=8 + more, prompt=300, step=19, depth=2, drafts=6, heads=(40, 8, 64), kv_dtype="bf16",
                                    q_dtype="bf16"),
    lambda more: sw.bfs_tot(n_queries=34 + more, prompt=75, step=30, width=4, keep=4, depth=1, heads=(71, 1, 64)),
    lambda more: sw.bfs_tot(n_queries=64 + more, prompt=40, step=20, width=16, keep=16, depth=1, heads=(16, 4, 64)),
    lambda more: _single_pieces(256 + more, heads=(40, 2, 128)),
    lambda more: _single_pieces(256 + more, heads=(40, 2, 64), kv_dtype="fp8_e4m3")])
@pytest.mark.parametrize("more", [0, 1])
def test_split_path_in_one_launch_and_in_phases(make, more):
    wl = make(more)
    assert_close(run_gpu(wl, kernel_mode=2), run_oracle_c(wl), wl.kv_dtype, wl.name)


# Items of more than 16 rows that are cut for phases but go in one launch, and beyond the bounds of 1536 workgroups (1024
# with heads of 64) in phases.
@pytest.mark.parametrize("make", [
    lambda more: sw.tot_with_drafts(n_queries=24 + more, prompt=75, step=19, depth=2, drafts=6, heads=(40, 8, 128), token_trees=True),
    lambda more: sw.tot_with_drafts(n_queries=12 + 8 * more, prompt=300, step=19, depth=2, drafts=6, heads=(40, 8, 64), kv_dtype="bf16",
                                    q_dtype="bf16"),
    lambda more: sw.bfs_tot(n_queries=68 + more, prompt=75, step=30, width=4, keep=4, depth=1, heads=(71, 1, 64)),
    lambda more: _single_pieces(768 + more, heads=(40, 2, 128)),
    lambda more: _single_pieces(512 + more, heads=(40, 2, 64), kv_dtype="fp8_e4m3")])
@pytest.mark.parametrize("more", [0, 1])
def test_items_of_two_row_tiles_together_and_in_phases(make, more):
    wl = make(more)
    assert_close(run_gpu(wl, kernel_mode=2), run_oracle_c(wl), wl.kv_dtype, wl.name)


# Short items of one page to 16, of whole and of partial blocks, fewer than run at a time (512 workgroups, 768 with heads of 64) and
# more: as row tiles, with one set of K and V registers, through LDS and, of the last, in phases.
@pytest.mark.parametrize("heads,kv_dtype", [((8, 2, 128), "fp8_e4m3"), ((8, 2, 64), "bf16"), ((12, 4, 64), "fp8_e4m3")])
@pytest.mark.parametrize("trees", [20, 50])
@pytest.mark.parametrize("step,chunk", [(1, 0), (33, 0), (250, 16), (280, 17), (100, 3)])
def test_many_short_items(heads, kv_dtype, trees, step, chunk):
    wl = sw.bfs_tot(n_queries=trees, prompt=21, step=step, width=8, keep=8, depth=1, heads=heads, kv_dtype=kv_dtype)
    got = run_gpu(wl, kernel_mode=2, prefix_chunk_pages=chunk, suffix_chunk_pages=chunk)
    assert_close(got, run_oracle_c(wl), kv_dtype, f"{heads} {kv_dtype} {trees} {step}")


@pytest.mark.parametrize("heads,kv_dtype", [((8, 2, 128), "fp8_e4m3"), ((8, 2, 64), "bf16")])
def test_many_short_items_with_draft_masks(heads, kv_dtype):
    wl = sw.tot_with_drafts(n_queries=100, prompt=40, step=19, depth=2, drafts=3, heads=heads, kv_dtype=kv_dtype, token_trees=True)
    assert_close(run_gpu(wl, kernel_mode=2), run_oracle_c(wl), kv_dtype, kv_dtype)


# The forms on either side of their bounds.  One set of registers: more items than run at a time, none of more than 64 rows,
# the longest of few rows and of branches 16 pages and not 17; row tiles of fp8: by number and length of the items; through LDS what is beyond, fp8
# groups of up to 64 and of up to 128 rows, one and both of the lists, at lengths given and at the planner's.
def _bfs(n, prompt, step, width, heads, kv_dtype="fp8_e4m3", keep=None, depth=1):
    return sw.bfs_tot(n_queries=n, prompt=prompt, step=step, width=width, keep=keep or width, depth=depth, heads=heads, kv_dtype=kv_dtype)


@pytest.mark.parametrize("make,chunks,form", [
    (lambda: _bfs(20, 21, 256, 16, (8, 2, 128)), (0, 16), ONE_REGISTER_SET), (lambda: _bfs(20, 21, 265, 16, (8, 2, 128)), (0, 17), THROUGH_LDS),
    (lambda: _bfs(13, 21, 256, 16, (12, 4, 64)), (0, 16), ONE_REGISTER_SET), (lambda: _bfs(13, 21, 265, 16, (12, 4, 64)), (0, 17), THROUGH_LDS),
    (lambda: _bfs(25, 21, 256, 16, (8, 2, 64), "bf16"), (0, 16), ONE_REGISTER_SET),
    (lambda: _bfs(25, 21, 265, 16, (8, 2, 64), "bf16"), (0, 17), THROUGH_LDS),
    (lambda: _bfs(24, 21, 40, 16, (8, 2, 128)), (0, 0), ONE_REGISTER_SET), (lambda: _bfs(70, 300, 40, 4, (8, 2, 128)), (0, 0), ONE_REGISTER_SET),
    (lambda: _bfs(30, 21, 100, 16, (8, 2, 64)), (0, 0), ONE_REGISTER_SET),
    (lambda: _bfs(40, 700, 20, 30, (8, 2, 128)), (0, 0), THROUGH_LDS),
    (lambda: _bfs(36, 200, 20, 32, (8, 2, 128), keep=2, depth=2), (0, 0), THROUGH_LDS),
    (lambda: _bfs(36, 200, 20, 32, (8, 2, 64), keep=2, depth=2), (0, 0), THROUGH_LDS),
    (lambda: _bfs(4, 6 * 384, 20, 24, (32, 8, 128)), (24, 0), ROW_TILES), (lambda: _bfs(4, 7 * 384, 20, 24, (32, 8, 128)), (24, 0), THROUGH_LDS),
    (lambda: _bfs(24, 5 * 384, 20, 16, (8, 2, 64)), (24, 0), ROW_TILES),
    (lambda: _bfs(24, 7 * 384, 20, 16, (8, 2, 64)), (24, 0), ONE_REGISTER_SET),
    (lambda: _bfs(8, 16, 20, 16, (8, 2, 128)), (0, 0), ROW_TILES), (lambda: _bfs(16, 16, 20, 16, (8, 2, 128)), (0, 0), ONE_REGISTER_SET)])
def test_forms_of_the_split_launch_at_their_bounds(make, chunks, form):
    wl = make()
    got = run_form(wl, form, prefix_chunk_pages=chunks[0], suffix_chunk_pages=chunks[1])
    assert_close(got, run_oracle_c(wl), wl.kv_dtype, f"{wl.name} {chunks}")


# Prompts shared by 17 to 128 rows and more, as row tiles of 16 and of 32 (20 heads a kv head) in a workgroup each: the last
# tile full, of one row and none at all (items of fewer rows than the list's span), chunks of one page, of a few and the planner's.
@pytest.mark.parametrize("heads,kv_dtype", [((8, 2, 128), "bf16"), ((8, 2, 64), "fp8_e4m3"), ((20, 1, 64), "bf16"), ((20, 1, 128), "fp8_e4m3"),
                                            ((17, 1, 128), "bf16")])
@pytest.mark.parametrize("width", [2, 5, 8, 9, 16, 17, 33])
@pytest.mark.parametrize("prompt,chunk", [(21, 0), (160, 3), (70, 1), (3001, 0)])
def test_items_of_many_rows_as_row_tiles(heads, kv_dtype, width, prompt, chunk):
    wl = sw.bfs_tot(n_queries=1, prompt=prompt, step=20, width=width, keep=width, depth=1, heads=heads, kv_dtype=kv_dtype)
    got = run_gpu(wl, kernel_mode=2, prefix_chunk_pages=chunk, suffix_chunk_pages=chunk)
    assert_close(got, run_oracle_c(wl), kv_dtype, f"{heads} {kv_dtype} {width} {prompt}")


# Either side of 512 row tiles, and of 992 with fp8 items of 3 pages and heads of 64: a prompt of 16 leaves takes 4 tiles of 16 rows
# a kv head and each leaf one, with drafts' masks the nodes of 4 leaves take 4 and 2 of 32 and each leaf one; beyond, the items go through LDS.
@pytest.mark.parametrize("kv_dtype,dim", [("bf16", 128), ("fp8_e4m3", 64)])
@pytest.mark.parametrize("drafts", [0, 5])
@pytest.mark.parametrize("n_queries", [12, 13, 24, 26, 27, 38, 39])
def test_items_of_many_rows_as_row_tiles_and_through_lds(kv_dtype, dim, drafts, n_queries):
    if drafts:
        wl = sw.tot_with_drafts(n_queries=n_queries, prompt=75, step=19, depth=2, drafts=drafts, heads=(10, 2, dim), kv_dtype=kv_dtype,
                                token_trees=True)
    else:
        wl = sw.bfs_tot(n_queries=n_queries, prompt=40, step=20, width=16, keep=16, depth=1, heads=(8, 2, dim), kv_dtype=kv_dtype)
    assert_close(run_gpu(wl, kernel_mode=2), run_oracle_c(wl), kv_dtype, f"{kv_dtype} {drafts} {n_queries}")


# A V page scale above 146 is read as 146 in nodes shared by more than 16 rows, whether few of them go as row tiles or many
# through LDS, bit for bit; in a branch of up to 16 rows it is read as given.
@pytest.mark.parametrize("heads,queries,width", [((8, 2, 128), 1, 8), ((8, 2, 64), 1, 8), ((20, 1, 128), 1, 3), ((8, 2, 128), 40, 32), ((8, 2, 64), 40, 32)])
def test_large_v_scales_of_nodes_shared_by_many_rows(heads, queries, width):
    import paper_2605_10195_amd as spex
    Hq, Hkv, D = heads
    rng = np.random.default_rng(3)

    def codes(n):
        return torch.from_numpy(rng.integers(0, 0x7F, size=(n, Hkv, D), dtype=np.uint8)).cuda()

    kr, vr, kb, vb = codes(40), codes(40), codes(20), codes(20)
    q = torch.from_numpy(rng.standard_normal((queries * width, Hq, D)).astype(np.float32)).to(torch.bfloat16).cuda()

    def run(root_scale, branch_scale):
        t = spex.SpexTree(Hq, Hkv, D, 16, "bf16", "fp8_e4m3", num_pages=queries * (3 + 2 * width), device="cuda", kernel_mode=2)
        ks = torch.full((3, Hkv), 1e-3, dtype=torch.float32, device="cuda")
        leaves = []
        for root in t.fork(-1, queries):
            t.append_step(root, kr, vr, ks, torch.full_like(ks, root_scale))
            for u in t.fork(root, width):
                t.append_step(u, kb, vb, ks[:2], torch.full_like(ks[:2], branch_scale))
                leaves.append(u)
        out, _ = t.decode_attention(leaves, None, q, D ** -0.5)
        torch.cuda.synchronize()
        t.close()
        return out

    want = run(146.0, 1.0)
    for scale in (147.0, 200.0, 1e4):
        assert torch.equal(run(scale, 1.0), want), scale
    if Hq // Hkv <= 16:
        # root values 0: the output is the branch's share, linear in its scale
        a, b = run(0.0, 100.0).double(), run(0.0, 400.0).double()
        assert float((b - 4 * a).norm() / b.norm()) <= 1e-6


@pytest.mark.parametrize("heads,kv_dtype,chunk", [((40, 2, 128), "bf16", 1), ((40, 2, 64), "fp8_e4m3", 2), ((34, 2, 128), "fp8_e4m3", 0)])
def test_phases_with_interior_nodes_and_cut_suffixes(heads, kv_dtype, chunk):
    """Requested nodes with and without live children, some twice, suffixes in one piece and in several."""
    wl = sw.random_trace(77, heads=heads, kv_dtype=kv_dtype, n_ops=900, n_roots=120, max_q_len=3)
    got = run_gpu(wl, kernel_mode=2, prefix_chunk_pages=chunk, suffix_chunk_pages=chunk)
    assert_close(got, run_oracle_c(wl), kv_dtype, f"{heads} chunk {chunk}")


def test_request_that_outgrows_its_plan_keeps_the_tree_walk_kernel():
    """160 long paths of one branch: the split path's estimate is lower, and its lists cannot follow a page that
    starts.  A request that outgrows its plan within 8 calls is planned for the tree-walk kernel, whose
    lists can; after 8 calls the estimate counts again."""
    import paper_2605_10195_amd as spex
    t = spex.SpexTree(4, 1, 64, 16, num_pages=160 * 390, device="cuda")
    roots = t.fork(-1, 160)
    for u in roots:
        t.append_step(u, None, None, n_tokens=6000)       # 375 whole pages
    t.k_pool.view(torch.bfloat16).normal_(0.0, 0.5)
    t.v_pool.view(torch.float16).normal_(0.0, 0.5)
    q = torch.randn((160, 4, 64), device="cuda").to(torch.bfloat16)

    def call(kernels):
        out, _ = t.decode_attention(roots, None, q, 0.125)
        assert (t.last_launch_info()["walk_row_tiles"] > 0) == (kernels == "walk")
        return out

    call("split")
    for u in roots:
        t.append_step(u, None, None, n_tokens=1)
    outs = [call("walk") for _ in range(9)]
    t.set_tuning(0, 0, 2, 0, 0)
    ref = call("split")
    assert float((outs[-1] - ref).norm() / ref.norm()) <= 1e-3
    t.set_tuning(0, 0, 0, 0, 0)
    for u in roots:
        t.append_step(u, None, None, n_tokens=200)
    call("split")
    t.close()
