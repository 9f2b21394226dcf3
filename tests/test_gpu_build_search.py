"""The searches of the index build at the edges of their tiles: list counts
around multiples of 32, token counts around multiples of a workgroup's 128 and
256, zero keys, both cache types and code widths. Every list and code of the
built index must be a nearest choice, in float64, under the model it exports,
and the first of equal ones."""

from __future__ import annotations

import pytest
import torch

from gpu_util import say
from paper_2609_33746_amd import pqhsa

pytestmark = pytest.mark.gpu

# Squared distances of vectors of norm at most 1 (2 for a residual) from sums
# of 128 products in 32 bits: 128 roundings of 2^-24 of a partial sum of at
# most 4.
TOL = 128 * 4 * 2.0 ** -24

CASES = [  # n_r, n_list, G heads, bits, dtype
    (255, 31, 1, 8, "bf16"),
    (256, 32, 1, 4, "bf16"),
    (257, 33, 2, 8, "bf16"),
    (1300, 97, 2, 4, "f32"),
    (127, 64, 1, 8, "f32"),
    (129, 1, 1, 8, "f32"),
    (3000, 1030, 1, 8, "bf16"),
]


@pytest.mark.parametrize("n_r,n_list,heads,bits,dtype", CASES)
def test_search_is_nearest(n_r, n_list, heads, bits, dtype):
    say(f"[build] n_r={n_r} n_list={n_list} heads={heads} bits={bits} {dtype}")
    m, ksub = (16, 256) if bits == 8 else (8, 16)
    n = n_r + 132
    gen = torch.Generator().manual_seed(n_r)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    key = torch.randn((1, heads, n, 128), generator=gen) * torch.empty((1, heads, n, 1)).uniform_(0.1, 9.0, generator=gen)
    key[:, :, 60] = 0.0                      # a zero key has the zero direction
    key[:, :, 80] = key[:, :, 70]            # and equal keys equal choices
    key = key.to(dt).cuda()
    val = torch.randn((1, heads, n, 128), generator=gen).to(dt).cuda()
    # more lists than tokens starts some centers on the same token: empty ones are re-seeded
    ic = torch.stack([4 + torch.randint(n_r, (n_list,), generator=gen) for _ in range(heads)])[None]
    ip = 4 + torch.randint(n_r, (1, heads, m, ksub), generator=gen)
    ctx = pqhsa.PQHSA(1, heads, heads, n, n_list, 16, kv_dtype=dtype, pq_m=m, pq_ksub=ksub)
    ctx.index_build([n], key, val, ic.to(torch.int32).cuda(), ip.to(torch.int32).cuda(), 1, 1)
    ix = ctx.index_export_tokens()
    for g in range(heads):
        k = key[0, g, 4:4 + n_r].double()
        r = torch.linalg.vector_norm(k, dim=1)
        assert torch.allclose(ix["norms"][0, g, 4:4 + n_r].double(), r, rtol=1e-6, atol=0)
        u = torch.where(r[:, None] > 0, k / r.clamp(min=1e-30)[:, None], torch.zeros_like(k))
        c = ix["centroids"][0, g].double()
        a = ix["list_ids"][0, g, 4:4 + n_r].long()
        d = torch.cdist(u, c, compute_mode="donot_use_mm_for_euclid_dist") ** 2
        assert float((d.gather(1, a[:, None])[:, 0] - d.min(1).values).max()) <= TOL
        assert int(a[80 - 4]) == int(a[70 - 4])
        res = (u - c[a]).view(n_r, m, 128 // m)
        for s in range(m):
            z = ix["codes"][0, g, 4:4 + n_r, s].long()
            d = torch.cdist(res[:, s].contiguous(), ix["codebooks"][0, g, s].double(),
                            compute_mode="donot_use_mm_for_euclid_dist") ** 2
            assert float((d.gather(1, z[:, None])[:, 0] - d.min(1).values).max()) <= TOL
            assert int(z[80 - 4]) == int(z[70 - 4])


def _build(key, val, n_list, bits, dtype, ic, ip, it_coarse, it_pq):
    m, ksub = (16, 256) if bits == 8 else (8, 16)
    b, heads, n, _ = key.shape
    ctx = pqhsa.PQHSA(b, heads, heads, n, n_list, 16, kv_dtype=dtype, pq_m=m, pq_ksub=ksub)
    ctx.index_build([n] * b, key, val, ic.to(torch.int32).cuda(), ip.to(torch.int32).cuda(), it_coarse, it_pq)
    return ctx.index_export_tokens()


def _bits(x):
    return x.contiguous().view(torch.int32) if x.dtype == torch.float32 else x


def _fma(a, b, c):
    """a b + c rounded once to 32 bits (the product is exact in float64)."""
    return (a.double() * b.double() + c.double()).float()


def _slices(ix, key, tokens, bits):
    """u = k / ||k|| and the residual slices u - c_a of the tokens, in 32 bits on the CPU, under the
    exported norms, lists and centroids: [tokens, 128] and [tokens, M, 128 / M]."""
    k = key[0, 0, tokens].float().cpu()
    r = ix["norms"][0, 0, tokens].cpu()
    u = k / r[:, None]
    res = u - ix["centroids"][0, 0].cpu()[ix["list_ids"][0, 0, tokens].cpu().long()]
    return u, res.view(len(tokens), 16 if bits == 8 else 8, -1)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_r,n_list,pairs,apart", [(3000, 64, 32, False), (2900, 129, 50, False),
                                                    (25000, 40, 1, False), (25000, 64, 32, True)])
def test_near_centers_are_the_choice_of_32_bit_sums(n_r, n_list, pairs, apart, dtype):
    """Centers in pairs of nearly one direction (the other ones ordinary; with one pair, all
    the others coincide): the list is the smallest ||c||^2 - 2 u . c of 32-bit sums in the
    order of the matrix instruction's steps, the first of equal ones. Every token is then a
    near tie, in the third case more of them than one round of its workgroups takes. With the
    pairs apart (by one bit of one element, or 1e-4 of each) the squared distances differ by
    about 1e-5: some tokens are near ties, and the others are up to the bf16 products alone
    (a CPU model of these without the product of the first center and second key part differs
    for 28 tokens in 32 bits, without the second and first for thousands in either type)."""
    say(f"[near centers] n_r={n_r} n_list={n_list} pairs={pairs} apart={apart} {dtype}")
    n = n_r + 132
    gen = torch.Generator().manual_seed(n_list)
    key = torch.randn((1, 1, n, 128), generator=gen)
    key = key.to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    even = key[:, :, 4:n - 1:2]
    if not apart:
        key[:, :, 5:n:2] = (3 if dtype == "bf16" else 1.2345) * even
    elif dtype == "bf16":
        bits = even.clone().view(torch.int16)
        x = torch.randint(128, (*bits.shape[:3], 1), generator=gen)
        key[:, :, 5:n:2] = bits.scatter(3, x, bits.gather(3, x) + 1).view(torch.bfloat16)
    else:
        key[:, :, 5:n:2] = even + 1e-4 * torch.randn(even.shape, generator=gen)
    pick = 4 + 2 * torch.randperm(n_r // 2, generator=gen)
    near = torch.stack([pick[:pairs], pick[:pairs] + 1], -1).flatten()
    rest = pick[pairs:pairs + n_list - 2 * pairs] if pairs > 1 else pick[1:2].expand(n_list - 2)
    ic = torch.cat([near, rest])[None, None]
    ip = pick[torch.arange(16 * 256) % 1000].view(1, 1, 16, 256)
    ix = _build(key.cuda(), key.cuda(), n_list, 8, dtype, ic, ip, 0, 0)
    t = torch.arange(4, 4 + n_r)
    u, _ = _slices(ix, key, t, 8)
    c = ix["centroids"][0, 0].cpu()
    q4 = c.view(n_list, 32, 4)
    sq = q4[:, :, 0] * q4[:, :, 0]
    for e in (1, 2, 3):
        sq = _fma(q4[:, :, e], q4[:, :, e], sq)
    while sq.shape[1] > 1:
        sq = sq[:, 0::2] + sq[:, 1::2]
    dot = torch.zeros((n_r, n_list))
    for x in [32 * q + j for j in range(32) for q in range(4)]:
        dot = _fma(u[:, x:x + 1], c[:, x][None], dot)
    want = _fma(torch.tensor(-2.0), dot, sq.T).numpy().argmin(1)
    got = ix["list_ids"][0, 0, t].cpu().numpy()
    assert (got == want).all(), int((got != want).sum())


NAN_CASES = [(8, "bf16"), (4, "f32"), (8, "f32"), (4, "bf16")]


@pytest.mark.parametrize("bits,dtype", NAN_CASES)
def test_a_key_with_a_nan_is_the_zero_direction(bits, dtype):
    """Rows that hold a NaN, of either sign, in one dimension or in all, have the
    norm NaN and otherwise count as zero keys: the index is bit for bit the one
    of the same keys with zeros in their place."""
    say(f"[nan] bits={bits} {dtype}")
    m, ksub = (16, 256) if bits == 8 else (8, 16)
    n_r, n_list, heads = 700, 20, 2
    n = n_r + 132
    gen = torch.Generator().manual_seed(bits)
    key = torch.randn((1, heads, n, 128), generator=gen)
    key = key.to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    val = torch.randn((1, heads, n, 128), generator=gen).to(key.dtype).cuda()
    ic = torch.stack([4 + torch.randperm(n_r, generator=gen)[:n_list] for _ in range(heads)])[None]
    ip = 4 + torch.randint(n_r, (1, heads, m, ksub), generator=gen)
    rows = [50, 51, 333]
    ip[0, :, :, 3] = rows[0]      # one of them also starts a codeword
    zero = key.clone()
    zero[:, :, rows] = 0.0
    nan = key.clone()
    nan[:, :, rows[0], 77] = float("nan")
    nan[:, :, rows[1], 5] = -torch.tensor(float("nan"), dtype=key.dtype)
    nan[:, :, rows[2]] = -torch.tensor(float("nan"), dtype=key.dtype)
    want = _build(zero.cuda(), val, n_list, bits, dtype, ic, ip, 1, 2)
    got = _build(nan.cuda(), val, n_list, bits, dtype, ic, ip, 1, 2)
    assert torch.isnan(got["norms"][:, :, rows]).all()
    got["norms"][:, :, rows] = want["norms"][:, :, rows]
    for name in ("list_means", "centroids", "codebooks"):
        assert torch.isfinite(got[name]).all(), name
        assert torch.equal(_bits(got[name]), _bits(want[name])), name
    for name in ("list_ids", "codes", "norms"):
        assert torch.equal(_bits(got[name][:, :, 4:4 + n_r]), _bits(want[name][:, :, 4:4 + n_r])), name


@pytest.mark.parametrize("bits,dtype", NAN_CASES)
def test_a_key_with_an_infinity(bits, dtype):
    """u = k / r of a row with an infinity is NaN there and 0 elsewhere: the row is
    in list 0, takes codeword 0 in the subspace of the infinity and makes that one
    dimension of that one codeword NaN, which no other token then chooses."""
    say(f"[inf] bits={bits} {dtype}")
    m, ksub = (16, 256) if bits == 8 else (8, 16)
    ds = 128 // m
    n_r, n_list, x, row = 700, 20, 77, 91
    n = n_r + 132
    gen = torch.Generator().manual_seed(10 + bits)
    key = torch.randn((1, 1, n, 128), generator=gen)
    key = key.to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    val = torch.randn((1, 1, n, 128), generator=gen).to(key.dtype).cuda()
    free = [t for t in range(4, 4 + n_r) if t != row]
    pick = torch.tensor(free)[torch.randperm(n_r - 1, generator=gen)]
    ic = pick[:n_list][None, None]
    ip = pick[torch.randint(n_r - 1, (1, 1, m, ksub), generator=gen)]
    key[:, :, row, x] = float("-inf")
    ix = _build(key.cuda(), val, n_list, bits, dtype, ic, ip, 0, 1)
    c = ix["centroids"][0, 0].double()
    cb = ix["codebooks"][0, 0].double()
    assert torch.isfinite(c).all()
    bad = torch.nonzero(torch.isnan(cb)).tolist()
    assert bad == [[x // ds, 0, x % ds]], bad
    assert int(ix["list_ids"][0, 0, row]) == 0 and int(ix["codes"][0, 0, row, x // ds]) == 0
    t = torch.tensor(free, device="cuda")
    k = key.cuda()[0, 0, t].double()
    u = k / torch.linalg.vector_norm(k, dim=1, keepdim=True)
    a = ix["list_ids"][0, 0, t].long()
    res = (u - c[a]).view(-1, m, ds)
    for s in range(m):
        z = ix["codes"][0, 0, t, s].long()
        d = torch.cdist(res[:, s].contiguous(), cb[s], compute_mode="donot_use_mm_for_euclid_dist") ** 2
        d = torch.nan_to_num(d, nan=float("inf"))
        assert float((d.gather(1, z[:, None])[:, 0] - d.min(1).values).max()) <= TOL


def _norms(k):
    """||k|| in 32 bits, 16 sums of 8 dimensions added in pairs."""
    x = k.float().view(-1, 16, 8)
    ss = torch.zeros(x.shape[:2])
    for e in range(8):
        ss = _fma(x[:, :, e], x[:, :, e], ss)
    while ss.shape[1] > 1:
        ss = ss[:, 0::2] + ss[:, 1::2]
    return torch.sqrt(ss[:, 0])


def _hard_rows(count, gen, dtype):
    """The rows of some 2^17 whose k / ||k|| lies closest to the middle of two 32-bit values."""
    k = torch.randn((1 << 17, 128), generator=gen).to(dtype)
    q = k.double() / _norms(k).double()[:, None]
    steps = q.abs() * torch.exp2(23.0 - torch.floor(torch.log2(q.abs().clamp(min=1e-30))))
    off = ((steps - torch.floor(steps)) - 0.5).abs().min(1).values
    return k[torch.argsort(off)[:count]]


@pytest.mark.parametrize("bits,dtype,size", [(8, "f32", 1.0), (4, "f32", 1.0), (8, "bf16", 1.0), (4, "bf16", 1.0),
                                             (8, "f32", 1e-6), (4, "f32", 1e-6)])
def test_a_codeword_of_one_token_is_its_residual(bits, dtype, size):
    """As many tokens as codewords, each the start of one: after a training pass every
    codeword is the mean of one residual, which is that residual bit for bit (the
    direction by an exactly rounded division, the sum without a step of its own)."""
    say(f"[one] bits={bits} {dtype} size={size}")
    m, ksub = (16, 256) if bits == 8 else (8, 16)
    n = ksub + 132
    gen = torch.Generator().manual_seed(3 * bits)
    key = size * torch.randn((1, 1, n, 128), generator=gen)
    if size < 1.0:   # directions of one large dimension: the residuals of the others are as small as they are
        key[..., 0] = 1.0
    key = key.to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    if size == 1.0:
        key[0, 0, 4:4 + ksub] = _hard_rows(ksub, gen, key.dtype)
    ic = torch.full((1, 1, 1), 4)
    ip = (4 + torch.arange(ksub)).expand(1, 1, m, ksub)
    ix = _build(key.cuda(), key.cuda(), 1, bits, dtype, ic, ip, 0, 1)
    _, res = _slices(ix, key, torch.arange(4, 4 + ksub), bits)
    for s in range(0 if size >= 1.0 else 1, m):
        assert torch.equal(_bits(ix["codebooks"][0, 0, s].cpu()), _bits(res[:, s].contiguous())), s


@pytest.mark.parametrize("bits,dtype", NAN_CASES)
def test_near_codewords_are_the_choice_of_32_bit_sums(bits, dtype):
    """Codewords in pairs that differ by the rounding of a direction, so that every token
    has two to choose from: the code is the smallest ||p||^2 - 2 r . p of a chain of
    32-bit fused multiply-adds over the dimensions (in the order of the matrix
    instruction's steps), the first of equal ones."""
    say(f"[near codewords] bits={bits} {dtype}")
    m, ksub = (16, 256) if bits == 8 else (8, 16)
    ds = 128 // m
    n_r, n_list = 3000, 12
    n = n_r + 132
    gen = torch.Generator().manual_seed(bits)
    key = torch.randn((1, 1, n, 128), generator=gen)
    key = key.to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    key[:, :, 5:n:2] = 1.2345 * key[:, :, 4:n - 1:2].float()   # pairs of tokens of nearly one direction
    if dtype == "bf16":
        key[:, :, 5:n:2] = 3 * key[:, :, 4:n - 1:2]            # a multiple that few bits of a key hold
    ic = 4 + 2 * torch.randperm(n_r // 2, generator=gen)[:n_list][None, None]
    first = 4 + 2 * torch.stack([torch.randperm(n_r // 2, generator=gen)[:ksub // 2] for _ in range(m)])
    ip = torch.stack([first, first + 1], -1).reshape(1, 1, m, ksub)
    ix = _build(key.cuda(), key.cuda(), n_list, bits, dtype, ic, ip, 0, 0)
    t = torch.arange(4, 4 + n_r)
    _, res = _slices(ix, key, t, bits)
    cb = ix["codebooks"][0, 0].cpu()
    order = [q * (ds // 4) + s for s in range(ds // 4) for q in range(4)]
    for s in range(m):
        p2 = torch.zeros(ksub)
        for x in range(ds):
            p2 = _fma(cb[s, :, x], cb[s, :, x], p2)
        dot = torch.zeros((n_r, ksub))
        for x in order:
            dot = _fma(res[:, s, x:x + 1], cb[s, :, x][None], dot)
        want = _fma(torch.tensor(-2.0), dot, p2[None]).numpy().argmin(1)
        got = ix["codes"][0, 0, t, s].cpu().numpy()
        assert (got == want).all(), (s, int((got != want).sum()))
