"""The update's encoding at the edges of its tiles (32 and 16 tokens, chunks of
64 centroids, shares of the centroids between workgroups): every new token's
list and codes must be a nearest choice in float64, a zero key has norm 0, and
the tokens already indexed stay."""

from __future__ import annotations

import pytest
import torch

from gpu_util import say
from paper_2609_33746_amd import pqhsa

pytestmark = pytest.mark.gpu

TOL = 128 * 4 * 2.0 ** -24   # 128 roundings of 2^-24 of a sum of at most 4

CASES = [  # new tokens, n_list, KV heads, bits, dtype
    (1, 1, 1, 8, "bf16"),
    (15, 63, 2, 8, "f32"),
    (16, 64, 1, 4, "bf16"),
    (17, 65, 3, 4, "f32"),
    (33, 300, 1, 8, "bf16"),
    (700, 1025, 2, 8, "bf16"),
    (9000, 40, 1, 8, "bf16"),   # more tokens than scratch for many shares
]


@pytest.mark.parametrize("new,n_list,heads,bits,dtype", CASES)
def test_encode_is_nearest(new, n_list, heads, bits, dtype):
    say(f"[update] new={new} n_list={n_list} heads={heads} bits={bits} {dtype}")
    m, ksub = (16, 256) if bits == 8 else (8, 16)
    old = 300
    n = old + new
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(new)
    f = dict(generator=gen, device="cuda")
    key = (3 * torch.randn((1, heads, n, 128), **f)).to(dt)
    key[:, :, old - 128] = 0.0               # the first new token
    val = torch.randn((1, heads, n, 128), **f).to(dt)
    cen = torch.nn.functional.normalize(torch.randn((1, heads, n_list, 128), **f), dim=-1)
    cb = 0.05 * torch.randn((1, heads, m, ksub, 128 // m), **f)
    ids = torch.randint(0, n_list, (1, heads, n), dtype=torch.int32, **f)
    codes = torch.randint(0, ksub, (1, heads, n, m), **f).to(torch.uint8)
    norms = torch.rand((1, heads, n), **f)
    means = torch.zeros((1, heads, n_list, 128), device="cuda")
    ctx = pqhsa.PQHSA(1, heads, heads, n, n_list, 16, kv_dtype=dtype, pq_m=m, pq_ksub=ksub)
    ctx.index_prepare([old], ids, codes, norms, cen, cb, means)
    ctx.index_update([n], key, val)
    ix = ctx.index_export_tokens()
    lo, mid, hi = 4, old - 128, n - 128
    for g in range(heads):
        assert torch.equal(ix["list_ids"][0, g, lo:mid], ids[0, g, lo:mid])
        assert torch.equal(ix["codes"][0, g, lo:mid], codes[0, g, lo:mid])
        k = key[0, g, mid:hi].double()
        r = torch.linalg.vector_norm(k, dim=1)
        assert torch.allclose(ix["norms"][0, g, mid:hi].double(), r, rtol=1e-6, atol=0)
        u = torch.where(r[:, None] > 0, k / r.clamp(min=1e-30)[:, None], torch.zeros_like(k))
        a = ix["list_ids"][0, g, mid:hi].long()
        d = torch.cdist(u, cen[0, g].double(), compute_mode="donot_use_mm_for_euclid_dist") ** 2
        assert float((d.gather(1, a[:, None])[:, 0] - d.min(1).values).max()) <= TOL
        res = (u - cen[0, g].double()[a]).view(-1, m, 128 // m)
        for s in range(m):
            z = ix["codes"][0, g, mid:hi, s].long()
            d = torch.cdist(res[:, s].contiguous(), cb[0, g, s].double(),
                            compute_mode="donot_use_mm_for_euclid_dist") ** 2
            assert float((d.gather(1, z[:, None])[:, 0] - d.min(1).values).max()) <= TOL
