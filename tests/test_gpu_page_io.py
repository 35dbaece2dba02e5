"""GPU: runs of tokens written into the pool and read back, byte for byte, over appends that start,
continue and end inside pages, more pages than one launch takes, and buffers that are not 16-byte
aligned (which take the element-wise kernels)."""

import pytest
import torch

from gpu_common import assert_v_round_trip

pytestmark = pytest.mark.gpu

KV = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8_e4m3": torch.uint8}
# tiled pools of both head dims, row-major ones (other page sizes, head dims, types), one whose rows
# are not a multiple of 16 bytes
SHAPES = [("bf16", 2, 128, 16), ("bf16", 3, 64, 16), ("fp8_e4m3", 2, 128, 16), ("fp8_e4m3", 5, 64, 16), ("bf16", 2, 40, 16),
          ("bf16", 2, 128, 64), ("f32", 2, 64, 16), ("f32", 1, 256, 4), ("fp8_e4m3", 2, 96, 32), ("fp8_e4m3", 2, 40, 8),
          ("bf16", 2, 20, 16), ("f32", 2, 7, 1)]


def draw(n, heads, dim, kv, seed, shift):
    """[n, heads, dim] tensor whose storage starts `shift` elements behind an aligned address."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    total = n * heads * dim
    if kv == "fp8_e4m3":
        x = torch.randint(0, 0x7F, (total + shift,), generator=g, device="cuda").to(torch.uint8)
    else:
        x = torch.randn((total + shift,), generator=g, device="cuda").to(KV[kv])
    return x[shift:].view(n, heads, dim)


@pytest.mark.parametrize("kv,heads,dim,page", SHAPES)
@pytest.mark.parametrize("runs,shift", [((1,), 0), ((16, 1, 31), 0), ((5, 3, 8, 17, 64), 0), ((7, 40), 1), ((140, 9), 0)])
@pytest.mark.parametrize("interleave", [False, True])
def test_appended_runs_come_back(kv, heads, dim, page, runs, shift, interleave):
    import paper_2605_10195_amd as spex
    total = sum(runs) * (16 if runs[0] == 140 and page == 16 else 1)   # 140 pages of 16: beyond one launch
    runs = [r * (16 if runs[0] == 140 and page == 16 else 1) for r in runs]
    n_pages = -(-total // page)
    t = spex.SpexTree(heads, heads, dim, page, "f32" if kv == "f32" else "bf16", kv, num_pages=n_pages + 3, device="cuda",
                      pool_fill=0xFF, interleave_kv=interleave)
    (u,) = t.fork(-1, 1)
    ks, vs, sk, sv, at = [], [], [], [], 0
    for i, n in enumerate(runs):
        k, v = draw(n, heads, dim, kv, 2 * i, shift), draw(n, heads, dim, kv, 2 * i + 1, shift)
        scales = (None, None)
        if kv == "fp8_e4m3":
            new = t.append_new_pages(u, n)
            scales = tuple(torch.rand((new, heads), device="cuda") + 0.5 + j for j in range(2))
            sk.append(scales[0])
            sv.append(scales[1])
        t.append_step(u, k, v, *scales)
        ks.append(k)
        vs.append(v)
        at += n
    want_k, want_v = torch.cat(ks), torch.cat(vs)
    for first, n in ((0, at), (at // 3, at - at // 3), (at - 1, 1)):
        k, v, gk, gv = t.gather_kv(u, first, n)
        assert torch.equal(k.view(KV[kv]), want_k[first:first + n])
        assert_v_round_trip(v.view(KV[kv]), want_v[first:first + n]) if (kv, page) == ("bf16", 16) and dim in (64, 128) else \
            _same(v.view(KV[kv]), want_v[first:first + n])
        if kv == "fp8_e4m3":
            pages = torch.arange(first, first + n, device="cuda") // page
            assert torch.equal(gk, torch.cat(sk)[pages]) and torch.equal(gv, torch.cat(sv)[pages])
    # slots behind the last token are zero in the pool (filled with 0xFF before), so that a kernel that
    # multiplies them by a weight of zero meets no NaN: the whole last page, less its tokens, per head
    last, left = t.path_pages(u)[0][-1], page - ((at - 1) % page + 1)
    size = page * dim * KV[kv].itemsize
    stride = heads * (2 if interleave else 1) * size
    for pool in (t.k_pool, t.v_pool):
        for h in range(heads):
            tile = pool[last * stride + h * size:last * stride + (h + 1) * size].view(KV[kv])
            assert int((tile == 0).sum()) >= left * dim
            assert not bool(torch.isnan(tile.float()).any())
    t.close()


def _same(got, want):
    assert torch.equal(got, want)


@pytest.mark.parametrize("heads,dim,page", [(2, 128, 16), (3, 64, 16), (2, 96, 32), (1, 256, 64), (2, 40, 8), (2, 20, 16)])
@pytest.mark.parametrize("runs,shift", [((1,), 0), ((16, 1, 31), 0), ((5, 3, 8, 17, 64), 0), ((7, 40), 1)])
def test_quantised_runs_give_the_oracle_codes(heads, dim, page, runs, shift):
    import numpy as np
    import paper_2605_10195_amd as spex
    from oracle.tree_attention import encode_e4m3
    t = spex.SpexTree(heads, heads, dim, page, "bf16", "fp8_e4m3", num_pages=-(-sum(runs) // page) + 2, device="cuda",
                      pool_fill=0xFF)
    (u,) = t.fork(-1, 1)
    at, want, scale = 0, ([], []), ({}, {})
    for i, n in enumerate(runs):
        pair = [draw(n, heads, dim, "bf16", 9 * i + j, shift) for j in range(2)]
        t.append_step(u, *pair, quantize=True)
        for j, x in enumerate(pair):
            x = x.float().cpu().numpy()
            for a in range(n):
                p = (at + a) // page
                if p not in scale[j]:                       # the tokens of this run in the page it starts
                    b = min(n, (p + 1) * page - at)
                    amax = np.abs(x[a:b]).max(axis=(0, 2)).astype(np.float32)
                    scale[j][p] = np.maximum(amax / np.float32(448.0), np.float32(2.0 ** -40))
                inv = np.float32(1.0) / scale[j][p]
                want[j].append(encode_e4m3((x[a] * inv[:, None]).ravel()).reshape(heads, dim))
        at += n
    k, v, sk, sv = t.gather_kv(u, 0, at)
    for got, s, j in ((k, sk, 0), (v, sv, 1)):
        assert np.array_equal(got.cpu().view(torch.uint8).numpy(), np.stack(want[j]))
        assert np.array_equal(s.cpu().numpy(), np.stack([scale[j][i // page] for i in range(at)]))
    t.close()


@pytest.mark.parametrize("kv,dim", [("f32", 8), ("bf16", 64)])
@pytest.mark.parametrize("phase", ["round and round", "longer lists", "two streams"])
def test_many_appends_in_flight(kv, dim, phase):
    """The lists of appended tokens lie in a ring of four segments of 16 calls that the kernels read while the host fills
    the next.  Behind a long kernel nothing runs until the host has gone round once; then it goes round four times more,
    or asks for longer segments while the lists of 16 calls wait, or takes two streams in turn."""
    import paper_2605_10195_amd as spex
    few, many, ring, page = 200, 700, 4 * 16, 16
    calls = 5 * ring
    t = spex.SpexTree(1, 1, dim, page, kv, kv, num_pages=few * -(-(calls + 2) // page) + many, device="cuda", pool_fill=0xFF)
    nodes = t.fork(-1, many)
    g = torch.Generator(device="cuda").manual_seed(1)
    k = torch.randn((calls + 1, many, 1, dim), generator=g, device="cuda").to(KV[kv])
    v = torch.randn((calls + 1, many, 1, dim), generator=g, device="cuda").to(KV[kv])
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    big = torch.randn((4096, 4096), device="cuda")
    big = big @ big * 1e-3                                    # loads the library before anything waits behind it
    at = {u: [] for u in range(many)}                         # tokens of every node, by the call that wrote them

    def append(i, n):
        t.append_tokens(nodes[:n], k[i, :n].contiguous(), v[i, :n].contiguous())
        for u in range(n):
            at[u].append(i)

    append(0, few)                                            # makes the ring
    torch.cuda.synchronize()
    with torch.cuda.stream(streams[0]):
        for _ in range(32):
            big = big @ big * 1e-3
        done = torch.cuda.Event()
        done.record()
    grow_at = 16 if phase == "longer lists" else calls + 1
    for i in range(1, calls + 1):
        if i == min(ring, grow_at):
            assert not done.query(), "the kernel in front ended before the ring was full"
        s = streams[i % 2 if phase == "two streams" else 0]
        for other in streams:
            s.wait_stream(other)
        with torch.cuda.stream(s):
            append(i, many if i == grow_at else few)
    torch.cuda.synchronize()
    for u in (0, 1, few - 1, few, many - 1):
        if not at[u]:
            continue
        got_k, got_v, _, _ = t.gather_kv(nodes[u], 0, len(at[u]))
        assert torch.equal(got_k, k[at[u], u])
        assert_v_round_trip(got_v, v[at[u], u]) if kv == "bf16" else _same(got_v, v[at[u], u])
    t.close()
