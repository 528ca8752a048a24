"""The compression where workgroups have sixteen waves (more than 4096 candidates and a CU for every
workgroup, or more than 16 384) and at the edges of their key registers, eight waves beside them, and
the in-place rounds at whole and broken rounds of every row size."""
import pytest
import torch

from tests.test_prefill_chunk_paths import test_in_place_chunk_matches_the_copying_way as in_place_chunk
from tests.test_select_branches import kept_by_sorting, test_select_branches as select_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,heads,heavy,recent,averaged,protect,tied", [
    (4097, 2, 300, 301, False, 0, False),      # 8 keys per thread of sixteen waves
    (8192, 3, 1024, 100, True, 0, True),
    (8193, 3, 1024, 100, False, 0, True),      # 16
    (16384, 1, 33, 2000, True, 0, False),
    (16385, 1, 33, 2000, False, 0, True),      # keys in LDS
    (40000, 2, 2000, 2096, False, 0, False),   # keys formed per sweep
    (4500, 260, 40, 25, False, 0, True),       # more workgroups than CUs: eight waves, 32 keys
    (9000, 2, 0, 500, False, 0, False),        # nothing competes
    (9000, 2, 500, 0, False, 0, True),
    (6000, 2, 64, 64, False, 1, True),         # a pattern
])
def test_selection_with_sixteen_waves(n, heads, heavy, recent, averaged, protect, tied):
    select_case(n, heads, heavy, recent, averaged, protect, tied)


@pytest.mark.parametrize("dt,d,heads,heavy,recent,chunks", [
    ("f16", 128, 2, 64, 64, (200, 150, 1)),        # one round of 128 slots
    ("f16", 128, 2, 100, 157, (257, 300)),         # two rounds and a slot
    ("bf16", 64, 2, 128, 128, (300, 256)),         # one round of 256
    ("bf16", 64, 3, 500, 269, (700, 900)),         # three and a slot
    ("f32", 128, 2, 32, 32, (80, 64, 90)),         # one round of 64
    ("f32", 128, 2, 1000, 25, (1100, 50)),         # sixteen and a slot; window within the chunk
    ("f16", 128, 2, 600, 2000, (3000, 100, 700)),  # a window longer than the chunk
])
def test_in_place_rounds(dt, d, heads, heavy, recent, chunks):
    in_place_chunk(dt, d, heads, heavy, recent, chunks, {})


@pytest.mark.parametrize("n,heads,heavy,recent,protect,tied", [
    (4097, 12, 400, 401, 0, True),             # workgroups per head that do not divide the CUs
    (16385, 12, 700, 333, 0, False),           # the same, keys in LDS
    (28672, 12, 1000, 1000, 0, True),
    (28673, 12, 1000, 1000, 0, False),         # the same, keys formed per sweep
    (28673, 40, 200, 57, 0, True),             # fewer workgroups than CUs: the scores stay in the L2
    (16384, 257, 100, 30, 0, False),           # more heads than CUs: eight waves, 32 keys, full
    (16385, 257, 100, 30, 0, True),            # sixteen waves, keys in LDS
    (28673, 257, 40, 25, 0, False),            # sixteen waves, keys formed per sweep
    (5000, 257, 60, 40, 1, False),             # a pattern, eight waves with keys in LDS
    (16384, 300, 60, 40, 1, True),
    (28673, 12, 700, 70, 1, False),            # a pattern, keys formed per sweep
])
def test_selection_over_many_heads(n, heads, heavy, recent, protect, tied):
    """Inputs are made on the device, rows compared as bit patterns."""
    from paper_2306_14048_amd import binding as hb
    dev, d, k = torch.device("cuda:0"), 64, heavy + recent
    g = torch.Generator(device=dev).manual_seed(n + heads)
    if tied:
        values = torch.tensor([0.0, 1e-40, 0.25, 0.5, 1.0, 7.0], device=dev)
        score = values[torch.randint(0, len(values), (heads, n), generator=g, device=dev)]
    else:
        score = torch.exp(1.5 * torch.randn(heads, n, generator=g, device=dev))
    K, V = (torch.randint(-2**15, 2**15, (1, heads, n, d), generator=g, device=dev, dtype=torch.int16) for _ in range(2))
    c = hb.H2OCache(1, heads, d, heavy, recent, torch.float16, device=dev, protect=protect, stride=97)
    c.prefill_select(K.view(torch.float16), V.view(torch.float16), score.view(1, heads, n))
    Kc, Vc, acc, pos = c.views()
    got = pos[0].cpu()
    rows = score.cpu()
    for h in range(heads):
        assert torch.equal(got[h].long(), kept_by_sorting(rows[h], heavy, recent, False, protect, 97)), h
    at = pos[0].long()
    assert torch.equal(acc[0].view(torch.int32), score.gather(1, at).view(torch.int32))
    for cached, full in ((Kc, K), (Vc, V)):
        assert torch.equal(cached[0].view(torch.int16), full[0].gather(1, at[..., None].expand(-1, -1, d)))
    c.close()


@pytest.mark.parametrize("dt,d,heads,heavy,recent,chunks", [
    ("f16", 64, 257, 30, 34, (4100, 4040)),        # more heads than CUs: eight waves, 32 keys
    ("f16", 64, 2, 100, 50, (8192, 8043, 100)),    # sixteen waves, 16 keys
    ("bf16", 64, 1, 200, 100, (16400, 200)),       # sixteen waves, keys in LDS
    ("f16", 64, 1, 60, 40, (29000, 50)),           # keys formed per sweep
])
def test_in_place_selection_branches(dt, d, heads, heavy, recent, chunks):
    in_place_chunk(dt, d, heads, heavy, recent, chunks, {})
