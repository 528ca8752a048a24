"""The prompt compression at the edges of its dispatch: where the ranking keys move from
8 to 32 registers per thread (4096 candidates), to LDS (16 384) and to being formed again
for every sweep (28 672), with one and with many workgroups per head.  Bit for bit
against a stable sort on the host (the kernel does no arithmetic but the rank value)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def kept_by_sorting(score, heavy, recent, averaged, protect, stride):
    """Ascending positions kept of one head's scores: what is protected for the last query,
    and the best of the rest (equal ones: the higher position) up to the budget."""
    n, k = len(score), heavy + recent
    pos = torch.arange(n)
    if n <= k:
        return pos
    rank = score / (n - pos).to(torch.float32) if averaged else score      # binary32 quotient
    t = n - 1
    if protect == 1:
        safe = (t - pos < recent) | ((t - pos) % stride == 0)
    else:
        safe = pos > t - recent
    if int(safe.sum()) > k:                    # covers more than the budget: its own best compete
        cand, keep, want = pos[safe], pos[:0], k
    else:
        cand, keep, want = pos[~safe], pos[safe], k - int(safe.sum())
    order = torch.sort(rank[cand], stable=True).indices                    # ties: position ascending
    best = cand[order[len(order) - want:]] if want else cand[:0]
    return torch.cat([keep, best]).sort().values


@pytest.mark.parametrize("n,heads,heavy,recent,averaged,protect,tied", [
    (4096, 3, 400, 401, False, 0, False),
    (4097, 3, 400, 401, True, 0, True),
    (513, 600, 33, 30, False, 0, True),        # one workgroup per head
    (16384, 2, 1700, 1577, False, 0, True),
    (16385, 2, 1700, 1577, True, 0, False),
    (28672, 1, 2048, 2048, False, 0, True),
    (28673, 1, 2048, 2048, False, 0, True),
    (28673, 30, 100, 103, False, 0, True),     # fewer workgroups per head: the scores stay in the L2
    (5000, 2, 300, 31, True, 1, True),
    (28673, 1, 300, 33, False, 1, True),
    (1531, 16, 153, 153, False, 0, False),     # heads in eights: a head's workgroups on one XCD
    (4097, 24, 400, 401, True, 0, True),
    (16384, 8, 1700, 1577, False, 0, False),
    (28673, 64, 700, 300, False, 0, True),
    (2500, 2, 0, 70, False, 0, False),         # window only
    (2500, 2, 70, 0, False, 0, True),          # no window
])
def test_select_branches(n, heads, heavy, recent, averaged, protect, tied):
    from paper_2306_14048_amd import binding as hb
    dev, d, k, stride = torch.device("cuda:0"), 64, heavy + recent, 97
    g = torch.Generator().manual_seed(n + heads)
    if tied:
        values = torch.tensor([0.0, 1e-40, 0.25, 0.5, 1.0, 7.0])
        score = values[torch.randint(0, len(values), (heads, n), generator=g)]
    else:
        score = torch.exp(1.5 * torch.randn(heads, n, generator=g))
    K = torch.randn(1, heads, n, d, generator=g).half()
    V = torch.randn(1, heads, n, d, generator=g).half()
    cache = hb.H2OCache(1, heads, d, heavy, recent, torch.float16, device=dev, rank=int(averaged),
                        protect=protect, stride=stride)
    cache.prefill_select(K.to(dev), V.to(dev), score.to(dev).view(1, heads, n))
    Kc, Vc, acc, pos = (x.cpu()[0] for x in cache.views())
    for h in range(heads):
        at = kept_by_sorting(score[h], heavy, recent, averaged, protect, stride)
        assert torch.equal(pos[h].long(), at), "head %d: kept positions differ" % h
        assert torch.equal(acc[h].view(torch.int32), score[h, at].view(torch.int32))
        assert torch.equal(Kc[h].view(torch.int16), K[0, h, at].view(torch.int16))
        assert torch.equal(Vc[h].view(torch.int16), V[0, h, at].view(torch.int16))
    cache.close()


@pytest.mark.parametrize("n", [700, 4097, 16385])          # eight waves; sixteen; keys in LDS
@pytest.mark.parametrize("digit", [0, 1, 2])
@pytest.mark.parametrize("spare", [0, 1])                  # the threshold's bin is kept whole, or all but one of it
def test_select_last_digit(n, digit, spare):
    """Scores that differ in one digit of the keys (11, 11 and 10 bits) only, at the ends and the middle of every
    wave's share of the bins: the threshold is found at that digit, in a bin of several equal scores."""
    from paper_2306_14048_amd import binding as hb
    dev, d, recent = torch.device("cuda:0"), 64, 20
    shift, bins = ((21, 1016), (10, 2048), (0, 1024))[digit]
    edges = torch.arange(0, bins, 64).repeat_interleave(3) + torch.tensor([0, 31, 63]).repeat(len(range(0, bins, 64)))
    edges = edges[edges < bins]                            # (below infinity)
    base = 0 if digit == 0 else 0x3f800000
    gen = torch.Generator().manual_seed(n + digit)
    cand = n - recent
    level = torch.randint(0, len(edges), (cand,), generator=gen)
    score = torch.cat([(base + (edges[level] << shift)).int().view(torch.float32), torch.zeros(recent)])
    from_top = torch.bincount(level, minlength=len(edges)).flip(0).cumsum(0)
    most = int(len(edges) * min(0.5, 3700 / n))            # (budgets end at 4096)
    for at in (most // 3, most):
        heavy = int(from_top[at]) - spare
        K = torch.randn(1, 8, n, d, generator=gen).half().to(dev)
        cache = hb.H2OCache(1, 8, d, heavy, recent, torch.float16, device=dev)
        cache.prefill_select(K, K, score.to(dev).expand(1, 8, n).contiguous())
        want = kept_by_sorting(score, heavy, recent, False, 0, 1)
        pos = cache.views()[3].cpu()[0].long()
        for h in range(8):
            assert torch.equal(pos[h], want), "head %d: kept positions differ" % h
        cache.close()
