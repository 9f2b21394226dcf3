"""The dense decode's splits: calls whose workgroup count moves the rows per
split between its bounds (128 and 4096), with lengths around a split's end and
ragged batches, against softmax attention in float64."""

from __future__ import annotations

import math

import pytest
import torch

from gpu_util import say
from paper_2609_33746_amd import pqhsa

pytestmark = pytest.mark.gpu

# name: (lengths, query heads, KV heads, dtype)
CASES = {
    "one-token": ([1], 4, 4, "bf16"),
    "shorter-than-a-split": ([127], 8, 1, "bf16"),
    "one-split": ([128], 4, 1, "f32"),
    "one-past": ([129], 4, 1, "bf16"),
    "half-splits": ([16383], 32, 8, "bf16"),
    "ragged-short": ([3000, 1, 2049], 16, 2, "f32"),
    "ragged-long": ([20001, 9000, 33, 15000, 20000, 12345, 4097, 4096], 32, 8, "bf16"),
    "longest-splits": ([9000, 4097] * 40, 8, 8, "bf16"),
}


@pytest.mark.parametrize("own", [False, True], ids=["noalloc", "context"])
@pytest.mark.parametrize("name", list(CASES))
def test_dense_splits(name, own):
    lens, hq, hkv, dtype = CASES[name]
    say(f"[dense] {name} own={own}")
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(len(name))
    n = max(lens)
    shape = (len(lens), hkv, n, 128)
    k = torch.randn(shape, generator=gen, device="cuda").to(dt)
    v = torch.randn(shape, generator=gen, device="cuda").to(dt)
    q = (2 * torch.randn((len(lens), hq, 128), generator=gen, device="cuda")).to(dt)
    for b, m in enumerate(lens):   # rows past a sequence's end must not be read into it
        k[b, :, m:] = float("nan")
        v[b, :, m:] = float("nan")
    if own:
        ctx = pqhsa.PQHSA(len(lens), hq, hkv, max(n, 132), 16, 16, kv_dtype=dtype)
        out = ctx.dense_decode(q, k, v, lens)
    else:
        out = pqhsa.dense_decode_noalloc(q, k, v, lens)
    G = hq // hkv
    for b, m in enumerate(lens):
        for g in range(hkv):
            p = torch.softmax(q[b, g * G:(g + 1) * G].double() @ k[b, g, :m].double().t() / math.sqrt(128), -1)
            want = p @ v[b, g, :m].double()
            # exponentials of logits up to about 40 in 32 bits: 40 roundings of 2^-24
            err = (out[b, g * G:(g + 1) * G].double() - want).abs().max() / want.abs().max()
            assert float(err) <= 40 * 2.0 ** -23, (b, g, float(err))
