"""The compression where workgroups have sixteen waves (more than 4096 candidates, one workgroup
per CU) and at the edges of their key registers, and the in-place rounds at whole and broken
rounds of every row size."""
import pytest
import torch

from tests.test_prefill_chunk_paths import test_in_place_chunk_matches_the_copying_way as in_place_chunk
from tests.test_select_branches import test_select_branches as select_case

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
