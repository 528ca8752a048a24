"""The 4-bit step at the edges of its dispatch (blocks of 64 slots, one to four per wave) and
of its fixed-point digits: queries whose elements span many orders of magnitude, logits
that overflow the shift, values with one huge row, and inputs that are not finite."""
import pytest
import torch

from tests.test_q4_parity import q4_case, torch_dt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,k,heads,dt", [
    (128, 63, 2, "f16"), (128, 64, 2, "bf16"), (128, 65, 2, "f16"),        # one block, two
    (128, 60, 520, "f16"),                                                 # one wave per head
    (128, 448, 2, "f16"), (128, 449, 2, "f16"), (128, 512, 2, "f32"),      # seven blocks; eight: two per wave
    (128, 513, 2, "bf16"), (128, 1025, 1, "f16"),                          # four per wave
    (64, 512, 2, "f16"), (64, 513, 2, "f16"), (64, 896, 2, "bf16"), (64, 897, 2, "f32"), (64, 2047, 1, "f16"),
])
def test_q4_block_edges(d, k, heads, dt):
    q4_case(1, heads, d, k + 3, 5, (k + 1) // 2, k // 2, torch_dt[dt], 1.0, 80 + k)
    if heads < 10:
        q4_case(1, heads, d, k - 3, 6, (k + 1) // 2, k // 2, torch_dt[dt], 1.0, 81 + k)   # fills, then evicts


@pytest.mark.parametrize("waves", range(1, 9))
def test_q4_shared_work_with_every_number_of_waves(waves):
    """Which wave sums, cuts digits and quantises the new token depends on how many there are."""
    k, heads = 64 * waves - 5, 520 if waves == 1 else 2          # (few heads: at least two waves)
    q4_case(1, heads, 64, k + 3, 4, (k + 1) // 2, k // 2, torch_dt["f16"], 1.0, 90 + waves)


@pytest.mark.parametrize("waves", [1, 2, 3, 8])
def test_q4_final_sums_of_binary32_elements(waves):
    """Two sums per wave, read of two waves where there are no more, else of eight."""
    k, heads = 64 * waves - 5, 520 if waves == 1 else 2
    q4_case(1, heads, 128, k + 3, 4, (k + 1) // 2, k // 2, torch_dt["f32"], 1.0, 190 + waves)


def dequantised(x):
    g = x.float().unflatten(-1, (-1, 64))
    mn, mx = g.amin(-1, keepdim=True), g.amax(-1, keepdim=True)
    sc = (mx - mn) / torch.full_like(mx, 15.0)
    code = torch.where(sc > 0, ((g - mn) / sc).round().clamp(0, 15), torch.zeros_like(g))
    return (mn.double() + code.double() * sc.double()).flatten(-2)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dt", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("kind", ["spread", "tiny", "above", "below", "one huge row"])
def test_q4_digits(dt, d, kind):
    """One step against float64 on the stored (dequantised) rows, on the CPU."""
    from paper_2306_14048_amd import binding as hb
    dev, dtype, heads, k = torch.device("cuda:0"), torch_dt[dt], 3, 150
    g = torch.Generator().manual_seed(len(kind) + d)
    rand = lambda *s: torch.randn(s, generator=g)  # noqa: E731
    K, V = rand(1, heads, k, d), rand(1, heads, k, d)
    q, kn, vn = rand(1, heads, d), rand(1, heads, d), rand(1, heads, d)
    if kind == "spread":                        # six orders of magnitude inside one query
        q = q * 10.0 ** (torch.randint(-5, 2, (1, heads, d), generator=g).float())
    elif kind == "tiny":
        q = q * 3e-5
    elif kind == "above":                       # logits some 2000 above the token's own
        q, kn, K = q.abs() + 1, torch.zeros_like(kn), K + (500 if d == 64 else 350) * (torch.arange(k) % 3 == 0)[:, None]
    elif kind == "below":
        q, kn, K = q.abs() + 1, torch.zeros_like(kn), K - 500
    else:
        V[:, :, 17] *= 1000.0
    K, V, q, kn, vn = (x.to(dtype) for x in (K, V, q, kn, vn))
    cache = hb.H2OCache(1, heads, d, k // 2, k // 2, dtype, device=dev, kv_bits=4)
    score = torch.rand(1, heads, k, generator=g)
    cache.prefill_select(K.to(dev), V.to(dev), score.to(dev))
    out = torch.empty(1, heads, d, dtype=dtype, device=dev)
    cache.decode_step(q.to(dev), kn.to(dev), vn.to(dev), out)
    acc = cache.views()[2].cpu()
    Kd, Vd = dequantised(K), dequantised(V)
    s = (Kd @ q.double().unsqueeze(-1)).squeeze(-1) * d ** -0.5
    own = (q.double() * kn.double()).sum(-1, keepdim=True) * d ** -0.5
    p = torch.softmax(torch.cat([s, own], -1), -1)
    ref = (p[..., None, :-1] @ Vd).squeeze(-2) + p[..., -1:] * vn.double()
    # one rounding of the probability to binary32 and one of its sum with the score
    want = (score.double() + p[..., :-1]).float()
    hit = (cache.views()[3].cpu() == k)                      # the slot that was given up
    assert int(hit.sum()) == heads
    assert bool(((acc.double() - want.double()).abs() <= 1.2e-7 * want.double()).logical_or(hit).all())
    # probabilities in binary32, then one rounding to the element type
    tol = {"f32": 3e-7, "f16": 2.0 ** -11 + 3e-7, "bf16": 2.0 ** -8}[dt]
    # (element by element: no slack from larger elements, groups or heads)
    size = (p[..., None, :-1] @ Vd.abs()).squeeze(-2) + p[..., -1:] * vn.double().abs()
    assert bool(((out.cpu().double() - ref).abs() <= tol * size).all())
    cache.close()


def q4_step(heads, d, dtype, K, V, q, kn, vn, scale=0.0):
    """One step on a 4-bit cache that holds all of K, V with zero scores and has room for the
    new token: (output, probability of every cached token and of the new one)."""
    from paper_2306_14048_amd import binding as hb
    dev, k = torch.device("cuda:0"), K.shape[2]
    cache = hb.H2OCache(1, heads, d, k, 1, dtype, scale, device=dev, kv_bits=4)
    cache.prefill_select(K.to(dev), V.to(dev), torch.zeros(1, heads, k, device=dev))
    out = torch.empty(1, heads, d, dtype=dtype, device=dev)
    cache.decode_step(q.to(dev), kn.to(dev), vn.to(dev), out)
    p = cache.views()[2].cpu().clone()
    cache.close()
    return out.cpu(), p


# Against the device's own (binary32) probabilities, element by element, the sums of |p v| as the
# measure: 16-bit elements have weights within 2^-30 of their group's largest in the block of 64
# slots (0.02 of the group's output here, times codes up to 15 and 410 slots: at most 1e-7),
# binary32 ones exact weights; then one rounding to the element type.
OUT_TOL = {"f32": 2.0 ** -24 * 1.01, "f16": 2.0 ** -11 + 1e-7, "bf16": 2.0 ** -8 + 1e-7}


@pytest.mark.parametrize("small", [0, 1])
@pytest.mark.parametrize("dt,ratio", [("f32", 1e3), ("f32", 1e5), ("f32", 1e9), ("bf16", 1e5), ("bf16", 1e9),
                                      ("f16", 3e5)])
def test_q4_value_groups_of_different_size(dt, ratio, small):
    """The values of one group of 64 elements are far smaller than those of the other: every
    group is as exact as if it were alone."""
    dtype, heads, k, d = torch_dt[dt], 3, 410, 128
    g = torch.Generator().manual_seed(int(ratio) + small)
    rand = lambda *s: torch.randn(s, generator=g)  # noqa: E731
    K, V, q, kn, vn = rand(1, heads, k, d), rand(1, heads, k, d), rand(1, heads, d), rand(1, heads, d), rand(1, heads, d)
    size_of = [ratio ** 0.5, ratio ** 0.5]                   # (f16: both ends stay normal numbers)
    size_of[small] = 1 / size_of[small]
    for x in (V, vn):
        x *= torch.tensor(size_of).repeat_interleave(64)
    check_output(dtype, dt, K, V, q, kn, vn)


@pytest.mark.parametrize("d,k", [(128, 410), (128, 1000), (64, 410), (64, 1000), (128, 2040)])
def test_q4_values_beside_a_dominant_row(d, k):
    """Binary32 elements, one token with nearly all the weight whose value row is zero in every
    second element: those elements come from the other tokens' weights of about 1e-9."""
    heads = 2
    g = torch.Generator().manual_seed(k + d)
    rand = lambda *s: torch.randn(s, generator=g)  # noqa: E731
    K, V, q, kn, vn = rand(1, heads, k, d), rand(1, heads, k, d).abs(), rand(1, heads, d), rand(1, heads, d), rand(1, heads, d)
    vn[..., 1::2] = 0.0
    V[:, :, 33, 1::2] = 0.0
    K[:, :, 33] = q * 20.0 / (q * q).sum(-1, keepdim=True) * d ** 0.5         # logit 20
    check_output(torch.float32, "f32", K, V, q, kn, vn)


def check_output(dtype, dt, K, V, q, kn, vn):
    K, V, q, kn, vn = (x.to(dtype) for x in (K, V, q, kn, vn))
    heads, d = q.shape[1], q.shape[2]
    out, p = q4_step(heads, d, dtype, K, V, q, kn, vn)
    Vd, p = dequantised(V), p.double()[..., None]
    ref = (p[..., :-1, :] * Vd).sum(-2) + p[..., -1, :] * vn.double()
    size = (p[..., :-1, :] * Vd.abs()).sum(-2) + p[..., -1, :] * vn.double().abs()
    if dt != "f32":
        size = size.unflatten(-1, (-1, 64)).amax(-1, keepdim=True).expand(-1, -1, -1, 64).flatten(-2)
    assert bool(((out.double() - ref).abs() <= OUT_TOL[dt] * size).all())


@pytest.mark.parametrize("dt", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("bad", [0, 1])
def test_q4_infinite_value_in_one_group(dt, bad):
    """An infinity in one group of a cached value row makes that group of the output not a
    number (a stored row has one scale per group) and leaves the other group as it is."""
    dtype, heads, k, d = torch_dt[dt], 2, 200, 128
    g = torch.Generator().manual_seed(7)
    rand = lambda *s: torch.randn(s, generator=g).to(dtype)  # noqa: E731
    K, V, q, kn, vn = rand(1, heads, k, d), rand(1, heads, k, d), rand(1, heads, d), rand(1, heads, d), rand(1, heads, d)
    want, _ = q4_step(heads, d, dtype, K, V, q, kn, vn)
    V[0, 0, 70, 64 * bad + 5] = float("inf")
    out, _ = q4_step(heads, d, dtype, K, V, q, kn, vn)
    good = 1 - bad
    assert bool(torch.isnan(out[0, 0, 64 * bad:64 * bad + 64]).all())
    assert torch.equal(out[0, 0, 64 * good:64 * good + 64], want[0, 0, 64 * good:64 * good + 64])
    assert torch.equal(out[0, 1], want[0, 1])


def test_q4_query_groups_of_different_size():
    """A query whose first 64 elements are 2^40 times the others, over keys whose sizes are the
    other way round: both groups count alike in a logit, and each keeps its digits."""
    heads, k, d = 3, 200, 128
    g = torch.Generator().manual_seed(11)
    rand = lambda *s: torch.randn(s, generator=g)  # noqa: E731
    K, V, q, kn, vn = rand(1, heads, k, d), rand(1, heads, k, d), rand(1, heads, d), rand(1, heads, d), rand(1, heads, d)
    q[..., :64] *= 2.0 ** 40
    for x in (K, kn):
        x[..., :64] *= 2.0 ** -40
    _, p = q4_step(heads, d, torch.float32, K, V, q, kn, vn)
    s = torch.cat([(dequantised(K) @ q.double().unsqueeze(-1)).squeeze(-1), (q.double() * kn.double()).sum(-1, keepdim=True)], -1)
    want = torch.softmax(s * d ** -0.5, -1)
    # one rounding to binary32 (the logits are exact to 1e-13)
    assert bool(((p.double() - want).abs() <= 6.1e-8 * want).all())


@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_q4_query_digits_round_to_nearest(dt):
    """Query elements a quarter of a digit unit below zero: each is off by at most half a unit
    (2^-54 for a largest element of 1), so the logit by at most 63 x 15 of them times the scale."""
    dtype, heads, k, d = torch_dt[dt], 1, 3, 64
    K = torch.full((1, heads, k, d), 15.0 * 2.0 ** 40)       # codes 15, scale 2^40 ...
    K[..., 0] = 0.0                                          # ... minimum 0
    q = torch.full((1, heads, d), -2.0 ** -55)
    q[..., 0] = 1.0
    kn = torch.zeros(1, heads, d)
    V, vn = torch.randn(1, heads, k, d), torch.randn(1, heads, d)
    K, V, q, kn, vn = (x.to(dtype) for x in (K, V, q, kn, vn))
    _, p = q4_step(heads, d, dtype, K, V, q, kn, vn, scale=1.0)
    logit = torch.log(p[0, 0, :k].double() / p[0, 0, k].double())
    true = (K.double() * q.double()[:, :, None]).sum(-1)[0, 0]
    assert float((logit - true).abs().max()) <= 63 * 15 * 2.0 ** -54 * 2.0 ** 40 * (1 + 1e-5) + 2e-7


def test_q4_not_finite():
    """An infinity in the query makes the head's output not a number; other heads are untouched."""
    from paper_2306_14048_amd import binding as hb
    dev, d, k = torch.device("cuda:0"), 128, 100
    g = torch.Generator().manual_seed(1)
    K, V = (torch.randn(1, 2, k, d, generator=g).half().to(dev) for _ in range(2))
    q, kn, vn = (torch.randn(1, 2, d, generator=g).half().to(dev) for _ in range(3))
    q[0, 1, 5] = float("inf")
    cache = hb.H2OCache(1, 2, d, 50, 50, torch.float16, device=dev, kv_bits=4)
    cache.prefill_select(K, V, torch.rand(1, 2, k, generator=g).to(dev))
    out = torch.empty(1, 2, d, dtype=torch.float16, device=dev)
    cache.decode_step(q, kn, vn, out)
    assert bool(torch.isfinite(out[0, 0]).all()) and bool(torch.isnan(out[0, 1]).all())
    cache.close()
