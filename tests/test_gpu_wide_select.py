"""The wide top-k select: rows of more than 1024 sub-chunks of 128 positions
(over 131072 indexed tokens), or whose budget leaves more candidates than the
plain select's LDS holds, against the oracle at the edges of its copy tiers
(8, 16 and 28 candidates per thread of 1024) and of its capacity."""

from __future__ import annotations

import pytest
import torch

from gpu_util import check_rows, context, make, run
from paper_2609_33746_amd import pqhsa, synth

pytestmark = pytest.mark.gpu

CAP = 28672      # candidate keys in LDS
FLOOD = -1_000_000   # a threshold bias that makes every token a candidate
STARVE = 1_000_000   # one that leaves none: the row is re-scanned

# name: (indexed tokens, k, threshold bias, variant)
CASES = {
    "1025-sub-chunks": (131073, 700, 0, "B"),
    "tier-8": (200001, 2000, 0, "B"),
    "tier-16": (400003, 4500, 0, "B"),
    "tier-28": (300007, 8000, 0, "B"),
    "k0": (140037, 0, 0, "B"),
    "k1": (140037, 1, 0, "C"),
    "bx": (160003, 4000, 0, "Bx"),
    "rescan": (140037, 300, STARVE, "B"),
    "all-tokens-past-capacity": (140037, 900, FLOOD, "B"),
    "large-budget-short-row": (CAP, 6000, 0, "B"),
    "all-tokens-at-capacity": (CAP, 6000, FLOOD, "B"),
    "all-tokens-one-past": (CAP + 1, 6000, FLOOD, "Bx"),
}


@pytest.mark.parametrize("name", list(CASES))
def test_wide_select(name):
    n_r, k, bias, variant = CASES[name]
    wl = synth.workload(1, batch=1, n_q_heads=4, n_kv_heads=1, max_seq=n_r + 132, n_list=300, topk=k)
    inp = make(wl, seed=23)
    ctx = context(inp)
    ctx.set_option(pqhsa.OPT_VARIANT, getattr(pqhsa, "VARIANT_" + variant.upper()))
    ctx.set_option(pqhsa.OPT_THRESHOLD_BIAS, bias)
    topk, out, sel, unsel, sc = run(ctx, inp, scores=True)
    check_rows(inp, topk, [(0, h) for h in range(4)], out, sel, unsel, sc, variant=variant)
    # the budget as device data: the wide select's other instantiation
    lens = inp["seq_lens"].to("cuda")
    got = ctx.decode_device_args(inp["q"], inp["k_cache"], inp["v_cache"], lens, inp["topk"].to("cuda"))
    assert torch.equal(got, out)
