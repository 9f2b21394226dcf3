"""The top-k select on long rows (over 131072 indexed tokens) and on rows whose
budget leaves more candidates than the plain select's LDS holds, which the wide
select takes: against the oracle at the edges of its copy tiers (8, 16 and 27
candidates per thread of 1024) and of its capacity."""

from __future__ import annotations

import pytest
import torch

from gpu_util import check_rows, context, make, run
from paper_2609_33746_amd import pqhsa, synth

pytestmark = pytest.mark.gpu

CAP = 27648      # candidate keys in LDS
FLOOD = -1_000_000   # a threshold bias that makes every token a candidate
STARVE = 1_000_000   # one that leaves none: the row is re-scanned

# name: (indexed tokens, k, threshold bias, variant)
CASES = {
    "long-row": (131073, 700, 0, "B"),
    "tier-8": (200001, 2000, 0, "B"),
    "tier-16": (400003, 4500, 0, "B"),
    "tier-27": (300007, 8000, 0, "B"),
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


@pytest.mark.parametrize("bits,n_r", [(4, 150001), (8, 150001), (8, 131072)],
                         ids=["pq4", "pq8-past-the-small-regions", "pq8-small-regions"])
def test_several_chunks_per_scan_workgroup(bits, n_r):
    """Grids of several scan rounds, where a workgroup scans several chunks:
    candidate regions of 2048 positions (4-bit codes, or over 1024 regions of
    128), or of 128."""
    kw = dict(batch=1, n_q_heads=16, n_kv_heads=16, max_seq=n_r + 132, topk=900)
    wl = synth.pq4(1, n_list=200, **kw) if bits == 4 else synth.workload(1, n_list=300, **kw)
    inp = make(wl, seed=29)
    ctx = context(inp)
    topk, out, sel, unsel, sc = run(ctx, inp, scores=True)
    check_rows(inp, topk, [(0, h) for h in (0, 7, 15)], out, sel, unsel, sc)
