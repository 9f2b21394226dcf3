"""The top-k select on long rows (over 131072 indexed tokens) and on rows whose
budget leaves more candidates than the plain select's LDS holds, which the wide
select takes: against the oracle at the edges of its copy tiers (8, 16 and 27
candidates per thread of 1024) and of its capacity. Every case names the capacity
that the call takes with the budgets on the host and as device data."""

from __future__ import annotations

import ctypes

import pytest
import torch

from gpu_util import check_rows, context, make, run
from paper_2609_33746_amd import pqhsa, synth

pytestmark = pytest.mark.gpu

SMALL, PLAIN, CAP = 7168, 12288, 27648      # candidates in LDS: two workgroups per CU, one, keys alone
FLOOD = -1_000_000   # a threshold bias that makes every token a candidate
STARVE = 1_000_000   # one that leaves none: the row is re-scanned

# name: (indexed tokens, k, threshold bias, variant, capacity, capacity with device budgets)
CASES = {
    "long-row": (131073, 700, 0, "B", PLAIN, PLAIN),
    "tier-8": (200001, 2000, 0, "B", PLAIN, PLAIN),
    "tier-16": (400003, 4500, 0, "B", CAP, CAP),
    "tier-27": (300007, 8000, 0, "B", CAP, CAP),
    "k0": (140037, 0, 0, "B", PLAIN, PLAIN),
    "k1": (140037, 1, 0, "C", PLAIN, PLAIN),
    "bx": (160003, 4000, 0, "Bx", PLAIN, PLAIN),
    "bx-wide": (300007, 6000, 0, "Bx", CAP, CAP),
    "bx-wide-host-only": (160003, 6000, 0, "Bx", CAP, PLAIN),
    "rescan": (140037, 300, STARVE, "B", PLAIN, PLAIN),
    "rescan-wide": (300007, 6000, STARVE, "B", CAP, CAP),
    "rescan-wide-bx": (300007, 6000, STARVE, "Bx", CAP, CAP),
    "all-tokens-past-capacity": (140037, 900, FLOOD, "B", PLAIN, PLAIN),
    "large-budget-short-row": (CAP, 6000, 0, "B", CAP, PLAIN),
    "all-tokens-at-capacity": (CAP, 6000, FLOOD, "B", CAP, PLAIN),
    "all-tokens-one-past": (CAP + 1, 6000, FLOOD, "Bx", CAP, PLAIN),
}


def _capacity(inp, topk, device_args):
    fn = pqhsa.load_library().pqhsa_select_capacity
    batch, n_q = inp["q"].shape[:2]
    ints = lambda v: (ctypes.c_int32 * batch)(*v)
    n_r = [int(n) - 132 for n in inp["seq_lens"]]
    return fn(batch, n_q, inp["centroids"].shape[2], max(topk), ints(n_r), ints(topk), int(device_args))


@pytest.mark.parametrize("name", list(CASES))
def test_wide_select(name):
    n_r, k, bias, variant, cap, cap_dev = CASES[name]
    wl = synth.workload(1, batch=1, n_q_heads=4, n_kv_heads=1, max_seq=n_r + 132, n_list=300, topk=k)
    inp = make(wl, seed=23)
    assert (_capacity(inp, [k], False), _capacity(inp, [k], True)) == (cap, cap_dev)
    ctx = context(inp)
    ctx.set_option(pqhsa.OPT_VARIANT, getattr(pqhsa, "VARIANT_" + variant.upper()))
    ctx.set_option(pqhsa.OPT_THRESHOLD_BIAS, bias)
    topk, out, sel, unsel, sc = run(ctx, inp, scores=True)
    check_rows(inp, topk, [(0, h) for h in range(4)], out, sel, unsel, sc, variant=variant)
    # the budget as device data
    lens = inp["seq_lens"].to("cuda")
    got = ctx.decode_device_args(inp["q"], inp["k_cache"], inp["v_cache"], lens, inp["topk"].to("cuda"))
    assert torch.equal(got, out)


@pytest.mark.parametrize("variant", ["B", "Bx"])
def test_wide_select_lowest_tier(variant):
    """A raised threshold that leaves about 6300 candidates for a budget of 4500:
    at most 8 per thread, in the wide select."""
    n_r, k = 400003, 4500
    wl = synth.workload(1, batch=1, n_q_heads=4, n_kv_heads=1, max_seq=n_r + 132, n_list=300, topk=k)
    inp = make(wl, seed=31)
    assert (_capacity(inp, [k], False), _capacity(inp, [k], True)) == (CAP, CAP)
    ctx = context(inp)
    ctx.set_option(pqhsa.OPT_VARIANT, getattr(pqhsa, "VARIANT_" + variant.upper()))
    sc = run(ctx, inp, scores=True)[4]
    top = torch.nan_to_num(sc[0], nan=float("-inf")).sort(dim=-1, descending=True).values
    usual = 2 * k + 8 * n_r // 2048      # the threshold's rank in tokens, but for the sample's spread
    bias = (top[:, 6300] - top[:, usual]).mean()
    ctx.set_option(pqhsa.OPT_THRESHOLD_BIAS, int(1000 * float(bias)))
    topk, out, sel, unsel, _ = run(ctx, inp)
    check_rows(inp, topk, [(0, h) for h in range(4)], out, sel, unsel, variant=variant)


@pytest.mark.parametrize("variant", ["B", "Bx"])
def test_wide_select_without_a_budget(variant):
    """A sequence with budget 0 beside one whose budget makes the call wide."""
    n_r, topk = 300007, [6000, 0]
    wl = synth.workload(1, batch=2, n_q_heads=2, n_kv_heads=1, max_seq=n_r + 132, n_list=300, topk=topk[0])
    inp = make(wl, seed=37)
    assert (_capacity(inp, topk, False), _capacity(inp, topk, True)) == (CAP, CAP)
    ctx = context(inp)
    ctx.set_option(pqhsa.OPT_VARIANT, getattr(pqhsa, "VARIANT_" + variant.upper()))
    topk, out, sel, unsel, _ = run(ctx, inp, topk=topk)
    check_rows(inp, topk, [(b, h) for b in range(2) for h in range(2)], out, sel, unsel, variant=variant)
    got = ctx.decode_device_args(inp["q"], inp["k_cache"], inp["v_cache"], inp["seq_lens"].to("cuda"),
                                 torch.tensor(topk, dtype=torch.int32, device="cuda"))
    assert torch.equal(got, out)


def test_small_select_at_two_percent():
    """264 rows of 128K tokens at 2%: about 5750 candidates a row, which two
    workgroups per CU hold."""
    n_r, k = 131072 - 132, 2621
    wl = synth.workload(1, batch=33, n_q_heads=8, n_kv_heads=1, max_seq=n_r + 132, n_list=1024, topk=k)
    inp = make(wl, seed=41)
    assert _capacity(inp, [k] * 33, False) == SMALL
    ctx = context(inp)
    topk, out, sel, unsel, _ = run(ctx, inp)
    check_rows(inp, topk, [(0, 0), (16, 3), (32, 7)], out, sel, unsel)


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
