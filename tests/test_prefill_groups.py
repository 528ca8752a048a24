"""Prompt attention where two wave groups share a block's keys, one phase apart and together: at
one tile, a tile and a row, a group without keys, and around the lines of the choice."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DT = {"f16": torch.float16, "bf16": torch.bfloat16}


@pytest.mark.parametrize("dt,d,heads,n", [
    ("f16", 128, 2, 480), ("f16", 128, 1, 512), ("bf16", 128, 2, 513), ("f16", 64, 3, 577), ("bf16", 64, 2, 640),
    ("f16", 128, 40, 768),        # 240 blocks: apart
    ("f16", 128, 43, 768),        # 258: together
    ("bf16", 64, 30, 1099),       # 270, below the line of the stream: together
    ("bf16", 128, 30, 1100),      # at it: apart
    ("f16", 64, 33, 860),         # 231 blocks in a grid of 280: apart
    ("bf16", 64, 50, 560),        # 250 in 280, a short stream: together
    ("f16", 64, 33, 1150),        # 297: apart
    ("bf16", 64, 36, 1100),       # 324 in 360: together
    ("f16", 64, 36, 1531),        # 432 in 480: apart
    ("f16", 64, 36, 1650),        # 468 in 520: together
    ("bf16", 64, 1, 9216),        # 72 in 576: apart
    ("f16", 64, 1, 9217),         # 73 in 584: together
])
def test_attention_rows_and_normalisers(dt, d, heads, n):
    from paper_2306_14048_amd import binding as hb
    g = torch.Generator(device="cuda").manual_seed(n + heads)
    Q, K, V = (torch.randn(1, heads, n, d, generator=g, device="cuda") for _ in range(3))
    K *= torch.exp(torch.randn(1, heads, n, 1, generator=g, device="cuda"))
    Q, K, V = (x.to(DT[dt]) for x in (Q, K, V))
    cfg = hb.make_config(1, heads, d, 8, 8, DT[dt])
    nb = hb.h2o_prefill_attention_workspace_bytes(cfg, n)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    out, lse = torch.empty_like(Q), torch.empty(heads, n, device="cuda")
    hb.h2o_prefill_attention(cfg, Q, K, V, n, ws, nb, out, lse)
    hidden = torch.ones(n, n, dtype=torch.bool, device="cuda").triu(1)
    # probabilities and outputs are rounded to the element type once each: half a unit of each
    tol = 2e-3 + (2 ** -8 if dt == "bf16" else 2 ** -11)
    for h in range(heads):
        s = (Q[0, h].float().double() @ K[0, h].double().t() / d ** 0.5).masked_fill(hidden, float("-inf"))
        ref = torch.softmax(s, -1) @ V[0, h].double()
        err = (out[0, h].double() - ref).norm(dim=-1) / ref.norm(dim=-1)
        assert float(err.max()) <= tol, "head %d: %g" % (h, float(err.max()))
        ref = torch.logsumexp(s, -1)
        assert torch.all((lse[h].double() - ref).abs() <= 1e-5 * (1 + ref.abs()))


@pytest.mark.parametrize("dt,heads,n", [
    ("f16", 2, 799), ("f16", 2, 800), ("bf16", 3, 833), ("f16", 1, 900), ("bf16", 36, 801), ("f16", 37, 897),
    ("f16", 13, 2500),            # 260 blocks, a long stream
])
def test_column_sums_of_groups_apart(dt, heads, n):
    from paper_2306_14048_amd import binding as hb
    g = torch.Generator(device="cuda").manual_seed(n)
    Q, K = (torch.randn(1, heads, n, 128, generator=g, device="cuda").to(DT[dt]) for _ in range(2))
    cfg = hb.make_config(1, heads, 128, 8, 8, DT[dt])
    got = hb.prefill_colsum(cfg, Q, K)[0].double()
    hidden = torch.ones(n, n, dtype=torch.bool, device="cuda").triu(1)
    for h in range(heads):
        s = (Q[0, h].double() @ K[0, h].double().t() / 128 ** 0.5).masked_fill(hidden, float("-inf"))
        ref = torch.softmax(s, -1).sum(0)
        assert torch.all((got[h] - ref).abs() <= 3e-5 * ref + 1e-30), "head %d" % h
