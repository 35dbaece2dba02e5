"""The form in which the split path launches the requests of tests/test_gpu_split_path.py, from plans made without a GPU: a
changed rule that empties one of those tests of the kernel it is for fails here."""

import pytest

import spex_workloads as sw

THROUGH_LDS, ONE_REGISTER_SET, ROW_TILES, IN_PHASES = range(4)  # SpexTree.split_form


def planned_form(wl, **kw):
    """The form that the split path takes for a workload, from a plan made without a GPU (draft masks do not change it)."""
    import paper_2605_10195_amd as spex
    t = spex.SpexTree(wl.num_q_heads, wl.num_kv_heads, wl.head_dim, wl.page_size, wl.q_dtype, wl.kv_dtype, num_pages=wl.peak_pages(),
                      device="cpu", **kw)
    sw.replay(wl, t, only_nodes=set())
    t.plan_dump(wl.leaves, wl.q_lens)
    form = t.split_form()
    t.close()
    return form


def test_many_short_items():
    for heads, kv_dtype in [((8, 2, 128), "fp8_e4m3"), ((8, 2, 64), "bf16"), ((12, 4, 64), "fp8_e4m3")]:
        for trees in (20, 50):
            for step, chunk in [(1, 0), (33, 0), (250, 16), (280, 17), (100, 3)]:
                wl = sw.bfs_tot(n_queries=trees, prompt=21, step=step, width=8, keep=8, depth=1, heads=heads, kv_dtype=kv_dtype)
                form = ROW_TILES if trees == 20 and step <= 250 and step != 100 else ONE_REGISTER_SET
                if (trees, step, kv_dtype) == (20, 280, "bf16"):
                    form = THROUGH_LDS
                if (trees, step, heads) == (50, 100, (12, 4, 64)):
                    form = IN_PHASES
                assert planned_form(wl, prefix_chunk_pages=chunk, suffix_chunk_pages=chunk) == form, (heads, kv_dtype, trees, step)


@pytest.mark.parametrize("heads,kv_dtype", [((8, 2, 128), "fp8_e4m3"), ((8, 2, 64), "bf16")])
def test_many_short_items_with_draft_masks(heads, kv_dtype):
    wl = sw.tot_with_drafts(n_queries=100, prompt=40, step=19, depth=2, drafts=3, heads=heads, kv_dtype=kv_dtype, token_trees=True)
    assert planned_form(wl) == ONE_REGISTER_SET


@pytest.mark.parametrize("heads,kv_dtype", [((8, 2, 128), "bf16"), ((8, 2, 64), "fp8_e4m3"), ((20, 1, 64), "bf16"), ((20, 1, 128), "fp8_e4m3"),
                                            ((17, 1, 128), "bf16")])
def test_items_of_many_rows_as_row_tiles(heads, kv_dtype):
    for width in (2, 5, 8, 9, 16, 17, 33):
        for prompt, chunk in [(21, 0), (160, 3), (70, 1), (3001, 0)]:
            wl = sw.bfs_tot(n_queries=1, prompt=prompt, step=20, width=width, keep=width, depth=1, heads=heads, kv_dtype=kv_dtype)
            few_rows, many_tiles = width * heads[0] // heads[1] <= 16, (heads[0], width, prompt) == (20, 33, 3001)
            form = planned_form(wl, prefix_chunk_pages=chunk, suffix_chunk_pages=chunk)
            assert form == (THROUGH_LDS if few_rows or many_tiles else ROW_TILES), (width, prompt)


@pytest.mark.parametrize("kv_dtype,dim", [("bf16", 128), ("fp8_e4m3", 64)])
@pytest.mark.parametrize("drafts", [0, 5])
def test_items_of_many_rows_as_row_tiles_and_through_lds(kv_dtype, dim, drafts):
    fp8_single = kv_dtype == "fp8_e4m3" and not drafts
    for n_queries in (12, 13, 24, 26, 27, 38, 39):
        if drafts:
            wl = sw.tot_with_drafts(n_queries=n_queries, prompt=75, step=19, depth=2, drafts=drafts, heads=(10, 2, dim), kv_dtype=kv_dtype,
                                    token_trees=True)
        else:
            wl = sw.bfs_tot(n_queries=n_queries, prompt=40, step=20, width=16, keep=16, depth=1, heads=(8, 2, dim), kv_dtype=kv_dtype)
        tiles = (24 if drafts else 40) * n_queries <= (992 if fp8_single else 512)
        assert planned_form(wl) == (ROW_TILES if tiles else ONE_REGISTER_SET if fp8_single else THROUGH_LDS), n_queries
