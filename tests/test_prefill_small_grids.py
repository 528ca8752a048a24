"""Column sums of binary32 prompts on small grids (blocks of 64 rows) at the edges of their tiles and on both sides of
every line of the rule (d = 64: 512 block slots; d = 128: 640, 32 tokens, two blocks per head beyond 128 heads and from 257
heads on up to 96 tokens), against float64.  Bar: the column sums' 3e-5 (three times the largest measured difference)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("heads,n", [(1, 1), (3, 32), (3, 33), (8, 63), (8, 64), (9, 65), (2, 127), (5, 129), (8, 1000),
                                     (64, 512), (64, 513), (64, 640), (64, 641), (65, 320), (65, 321), (128, 128), (129, 65),
                                     (192, 129), (200, 129), (264, 96), (264, 97), (512, 32), (512, 33)])
def test_binary32_column_sums_of_small_grids(d, heads, n):
    from paper_2306_14048_amd import binding as hb
    dev = torch.device("cuda:0")
    g = torch.Generator().manual_seed(n + heads)
    Q, K, V = (torch.randn(1, heads, n, d, generator=g).to(dev) for _ in range(3))
    col = torch.empty(1, heads, n, device=dev)
    cache = hb.H2OCache(1, heads, d, 8, 8, torch.float32, device=dev)
    cache.prefill_scores(Q, K, V, colsum_out=col)
    logits = torch.matmul(Q.double(), K.double().transpose(-1, -2).contiguous()) / d ** 0.5
    logits.masked_fill_(torch.ones(n, n, dtype=torch.bool, device=dev).triu(1), -torch.inf)
    want = torch.softmax(logits, -1).sum(-2)
    assert bool(((col - want).abs() <= 3e-5 * want).all())
    cache.close()
