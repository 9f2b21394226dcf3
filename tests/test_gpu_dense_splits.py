"""The dense decode's splits: calls whose workgroup count moves the rows per
split between its bounds (128 and 2048), with lengths around a split's end,
ragged batches and rows of up to 323 partials, against softmax attention in
float64."""

from __future__ import annotations

import ctypes
import math

import pytest
import torch

from gpu_util import say
from paper_2609_33746_amd import pqhsa

pytestmark = pytest.mark.gpu

# name: (lengths, query heads, KV heads, dtype, rows per split on 256 CUs)
CASES = {
    "one-token": ([1], 4, 4, "bf16", 128),
    "shorter-than-a-split": ([127], 8, 1, "bf16", 128),
    "one-split": ([128], 4, 1, "f32", 128),
    "one-past": ([129], 4, 1, "bf16", 128),
    "half-splits": ([16383], 32, 8, "bf16", 256),
    "ragged-short": ([3000, 1, 2049], 16, 2, "f32", 128),
    "ragged-long": ([20001, 9000, 33, 15000, 20000, 12345, 4097, 4096], 32, 8, "bf16", 864),
    "longest-splits": ([9000, 4097] * 40, 8, 8, "bf16", 928),
    # one KV head: 249 partials a row, and more than a merge takes in one round trip
    "one-head": ([135000], 8, 1, "bf16", 544),
    "one-head-longest": ([660000], 8, 1, "bf16", 2048),
    "four-per-cu": ([65536], 64, 8, "bf16", 512),
    "one-per-cu": ([20000, 20000], 16, 4, "f32", 640),
    "doubled": ([2900, 2049, 1600, 2800] * 8, 16, 4, "f32", 736),
    "no-longer-than-2048": ([4096] * 128, 8, 4, "bf16", 2048),
}


def _rule(lens, hq, hkv, dtype, partials):
    fn = pqhsa.load_library().pqhsa_dense_split_rows
    return fn(len(lens), hq, hkv, int(dtype == "bf16"), (ctypes.c_int32 * len(lens))(*lens), ctypes.c_int64(partials))


SPARE = 1 << 30
RULE = [  # equal lengths: a whole number of workgroups per CU, or the buffer's own splits
    ([131072], 32, 8, "bf16", SPARE, 2048),
    ([131072], 64, 8, "bf16", SPARE, 1024),
    ([65536], 32, 8, "f32", SPARE, 2048),
    ([50001] * 4, 32, 8, "bf16", SPARE, 1568),
    ([150000] * 8, 8, 2, "f32", SPARE, 1888),
    ([150000] * 8, 8, 2, "f32", 8 * 8 * 74, 2048),
    ([131072] * 16, 32, 8, "bf16", SPARE, 2048),
    ([1 << 20], 8, 1, "bf16", SPARE, 2048),
    ([30000, 15001] * 4, 64, 8, "bf16", 8192, 1888),
]


@pytest.mark.parametrize("lens,hq,hkv,dtype,partials,rows", RULE)
def test_rows_per_split(lens, hq, hkv, dtype, partials, rows):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("rows of 256 CUs")
    assert _rule(lens, hq, hkv, dtype, partials) == rows


@pytest.mark.parametrize("own", [False, True], ids=["noalloc", "context"])
@pytest.mark.parametrize("name", list(CASES))
def test_dense_splits(name, own):
    lens, hq, hkv, dtype, rows = CASES[name]
    say(f"[dense] {name} own={own}")
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert _rule(lens, hq, hkv, dtype, SPARE) == rows
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
