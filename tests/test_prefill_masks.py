"""Column sums at the sizes where a tile needs the causal mask, the end of the prompt, both or
neither, against float64; and rows that are not numbers, which only reach the keys they see."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


def column_sums(Q, K, first=0):
    """float64 column sums of the causal softmax; query row i sits at key position first + i."""
    n, m = K.shape[-2], Q.shape[-2]
    s = Q.double() @ K.double().transpose(-1, -2) / Q.shape[-1] ** 0.5
    hidden = torch.ones(m, n, dtype=torch.bool).triu(first + 1)
    return torch.softmax(s.masked_fill(hidden, float("-inf")), -1).sum(-2)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dt", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("heads", [2, 150])
def test_column_sums_at_tile_edges(heads, dt, d):
    from paper_2306_14048_amd import binding as hb
    g = torch.Generator().manual_seed(d + heads)
    sizes = (1, 31, 32, 33, 64, 65, 97, 128, 129, 191, 256, 257, 300, 511, 640) if heads == 2 else (33, 130, 256, 290)
    for n in sizes:
        Q, K = (torch.randn(1, heads, n, d, generator=g).to(DT[dt]) for _ in range(2))
        cfg = hb.make_config(1, heads, d, 8, 8, DT[dt])
        got = hb.prefill_colsum(cfg, Q.cuda(), K.cuda()).cpu().double()
        ref = column_sums(Q, K)
        # 32-bit sums and exponentials of logits below 2^5: a few 2^-24 each, as the other bars
        assert torch.all((got - ref).abs() <= 3e-5 * ref.abs() + 1e-30), "n = %d" % n


@pytest.mark.parametrize("dt,d", [("f32", 128), ("f16", 128), ("bf16", 64)])
@pytest.mark.parametrize("n,row", [(100, 40), (290, 129), (64, 63)])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_a_row_that_is_no_number_reaches_the_keys_it_sees(dt, d, n, row, value):
    from paper_2306_14048_amd import binding as hb
    g = torch.Generator().manual_seed(n)
    Q, K = (torch.randn(1, 1, n, d, generator=g).to(DT[dt]) for _ in range(2))
    Q[0, 0, row, 3] = value
    cfg = hb.make_config(1, 1, d, 8, 8, DT[dt])
    got = hb.prefill_colsum(cfg, Q.cuda(), K.cuda()).cpu()[0, 0]
    assert torch.isnan(got[:row + 1]).all()
    ref = column_sums(Q[:, :, row + 1:], K, row + 1)[0, 0, row + 1:]
    assert torch.all((got[row + 1:].double() - ref).abs() <= 3e-5 * ref + 1e-30)
