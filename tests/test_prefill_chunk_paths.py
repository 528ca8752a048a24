"""A chunk on a cache whose slots are in position order (cached rows used in place, the
compression moves rows inside the cache) against the way that copies cache and chunk
together first, which a restored cache takes: bit for bit, after every chunk."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


@pytest.mark.parametrize("dt,d,heads,heavy,recent,chunks,more", [
    ("f16", 128, 3, 100, 93, (300, 1, 64, 63, 257, 130), {}),          # ragged, single tokens, whole tiles
    ("bf16", 128, 2, 410, 409, (1024, 1000, 24), {}),
    ("bf16", 64, 3, 700, 600, (500, 600, 700, 100), {}),               # fills up first (nothing moves)
    ("f32", 128, 2, 65, 64, (129, 200, 3), {}),
    ("f32", 64, 2, 33, 30, (64, 64, 64), {}),
    ("f16", 64, 2, 40, 0, (100, 100), {}),                             # no window
    ("f16", 128, 2, 0, 64, (100, 64, 10), {}),                         # window only: every row moves
    ("bf16", 128, 2, 60, 61, (150, 150), dict(rank=1)),
    ("f16", 128, 2, 150, 20, (400, 333), dict(protect=1, stride=7)),
    ("f16", 128, 2, 2048, 2048, (4200, 1500), {}),                     # sixteen waves, 8 keys
    ("bf16", 128, 160, 256, 256, (600, 2048), {}),                     # column sums with eight waves
    # several workgroups per head, with some columns of its rows each (128 KiB of keys on)
    ("f16", 128, 8, 256, 256, (700, 3, 513), {}),                      # 4, at the line
    ("f16", 128, 9, 256, 255, (700, 300), {}),                         # one, below it
    ("f32", 128, 3, 300, 300, (700, 333, 1), {}),                      # 4 of 8
    ("f32", 128, 2, 700, 801, (2000, 600), {}),                        # 8
    ("f16", 64, 33, 512, 512, (1100, 500), dict(rank=1)),              # 2
    ("bf16", 128, 65, 300, 400, (800, 300), {}),                       # 2 (heads)
    ("f16", 128, 5, 800, 100, (1000, 777), dict(protect=1, stride=5)),
    ("bf16", 128, 2, 0, 900, (1000, 300, 901), {}),                    # window only
    ("bf16", 128, 16, 700, 500, (900, 700, 5000), {}),                 # fills up first; sixteen waves
    ("f16", 128, 2, 300, 300, (700, 17000), {}),                       # sixteen waves, keys in LDS
    ("bf16", 128, 3, 300, 300, (700, 29000), {}),                      # ... keys formed per sweep, from scores read again
    ("f16", 128, 2, 500, 100, (700, 17000, 29000), dict(protect=1, stride=37)),
    ("f32", 64, 9, 400, 200, (700, 29000), dict(rank=1)),
])
def test_in_place_chunk_matches_the_copying_way(dt, d, heads, heavy, recent, chunks, more):
    from paper_2306_14048_amd import binding as hb
    dev, dtype = torch.device("cuda:0"), DT[dt]
    g = torch.Generator().manual_seed(sum(chunks) + d)
    a, b = (hb.H2OCache(1, heads, d, heavy, recent, dtype, device=dev, **more) for _ in range(2))
    for i, m in enumerate(chunks):
        Q, K, V = (torch.randn(1, heads, m, d, generator=g).to(dtype).to(dev) for _ in range(3))
        K *= 2
        outs = [torch.zeros_like(Q) if dt != "f32" else None for _ in range(2)]
        a.prefill_chunk(Q, K, V, out=outs[0])
        if i:                                     # a restored cache: slot order is not known
            b.restore(*(x.clone() for x in b.views()), b.tokens_seen)
        b.prefill_chunk(Q, K, V, out=outs[1])
        torch.cuda.synchronize()
        (Ka, Va, aa, pa), (Kb, Vb, ab, pb) = a.views(), b.views()
        occ = pa >= 0
        assert torch.equal(pa, pb), "chunk %d: kept positions differ" % i
        assert torch.equal(aa.view(torch.int32), ab.view(torch.int32))
        assert torch.equal(Ka[occ].view(torch.uint8), Kb[occ].view(torch.uint8))
        assert torch.equal(Va[occ].view(torch.uint8), Vb[occ].view(torch.uint8))
        if outs[0] is not None:
            assert torch.equal(outs[0], outs[1])
    a.close()
    b.close()


def test_chunk_output_over_its_values():
    from paper_2306_14048_amd import binding as hb
    dev = torch.device("cuda:0")
    g = torch.Generator().manual_seed(3)
    a, b, c = (hb.H2OCache(1, 2, 128, 50, 50, torch.float16, device=dev) for _ in range(3))
    for m in (130, 140):
        Q, K, V = (torch.randn(1, 2, m, 128, generator=g).half().to(dev) for _ in range(3))
        out, over_v, over_k = torch.empty_like(Q), V.clone(), K.clone()
        a.prefill_chunk(Q, K, V, out=out)
        b.prefill_chunk(Q, K, over_v, out=over_v)
        c.prefill_chunk(Q, over_k, V, out=over_k)
        torch.cuda.synchronize()
        assert torch.equal(out, over_v) and torch.equal(out, over_k)
        for x in (b, c):
            assert all(torch.equal(y, z) for y, z in zip(a.views(), x.views()))
    for x in (a, b, c):
        x.close()


@pytest.mark.parametrize("what", ["output", "chunk"])
def test_chunk_over_the_cache_memory(what):
    """A chunk whose output goes over the cache's rows, or whose keys and values are read from
    there: the new state is what separate buffers give."""
    from paper_2306_14048_amd import binding as hb
    dev, d, heads, m = torch.device("cuda:0"), 128, 2, 90
    g = torch.Generator().manual_seed(5)
    rand = lambda n: torch.randn(1, heads, n, d, generator=g).half().to(dev)  # noqa: E731
    a, b = (hb.H2OCache(1, heads, d, 60, 60, torch.float16, device=dev) for _ in range(2))
    first = [rand(200) for _ in range(3)]
    for c in (a, b):
        c.prefill_chunk(*first, out=torch.empty_like(first[0]))
    Q, K, V = (rand(m) for _ in range(3))
    out = torch.empty_like(Q)
    lie = [x.reshape(-1)[:heads * m * d].view(1, heads, m, d) for x in b.views()[:2]]
    if what == "output":
        a.prefill_chunk(Q, K, V, out=out)
        b.prefill_chunk(Q, K, V, out=lie[0])
    else:
        a.prefill_chunk(Q, lie[0].clone(), lie[1].clone(), out=out)
        over = torch.empty_like(Q)
        b.prefill_chunk(Q, lie[0], lie[1], out=over)
        assert torch.equal(out, over)
    assert all(torch.equal(x, y) for x, y in zip(a.views(), b.views()))
    a.close()
    b.close()
