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
