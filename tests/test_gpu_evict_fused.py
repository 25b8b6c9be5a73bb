"""bkv_evict as one launch (bf16 fast path: score, selection and compaction
work items of every head under one ticket) and as the chained calls inside it,
against the oracle and against the chained entry points.

Checks per case:
  * scores within 1e-3 of the oracle;
  * isolation, zero tolerance: the oracle's selection fed the GPU's own
    scores gives exactly the GPU's kept indices, and the oracle's compaction
    fed the GPU's kept indices gives exactly the GPU's K and V;
  * bkv_score -> bkv_topk -> bkv_compact on a copy give the same kept
    indices and the same K and V bit for bit.
The fused launch takes large layers only (FUSED, which asserts that it does);
CHAINED are small ones of every shape.  Cases cover ragged N, N_cap > N,
D = 64, the prefix, W = 0, C = 0, N <= budget, rows in several register groups
(also four, one per wave), the scoring options, outputs left to the workspace,
and layers whose keys repeat a few rows only, so that scores tie in bulk (the
selection's exact radix path and its tie ranking by index)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_scores_close, dims_of, host, raw_bits, say
from score_layout import fuses
import paper_2609_04971_amd as bkv
from paper_2609_04971_amd import synth

pytestmark = pytest.mark.gpu

W = synth.Workload
# layers for the chained calls inside bkv_evict, many of the fused launch's own
# head lengths; "many-heads" is large enough for the fused launch
CHAINED = {
    "ragged": W("f1", B=2, Hq=8, Hkv=2, D=128, N=20001, W=8, C=4, budget=3000, revisit_frac=0.1),
    "prefix": W("f2", B=2, Hq=8, Hkv=2, D=128, N=16384, W=16, C=8, budget=2000, n_prefix=5),
    "d64-g7": W("f3", B=1, Hq=14, Hkv=2, D=64, N=17000, W=5, C=3, budget=2048, n_centroids=3),
    "no-window": W("f4", B=1, Hq=8, Hkv=2, D=128, N=16500, W=0, C=8, budget=1000),
    "n-below-budget": W("f5", B=1, Hq=4, Hkv=2, D=128, N=16384, W=8, C=4, budget=20000),
    "n-equals-budget": W("f6", B=1, Hq=4, Hkv=2, D=128, N=16384, W=8, C=4, budget=16384),
    "two-row-groups": W("f7", B=1, Hq=14, Hkv=2, D=128, N=16384, W=24, C=16, budget=1500, n_centroids=16),
    "many-heads": W("f8", B=16, Hq=32, Hkv=8, D=128, N=16384, W=32, C=16, budget=2048, revisit_frac=0.05),
    "32k": W("f9", B=1, Hq=8, Hkv=2, D=128, N=32768, W=32, C=16, budget=4096, revisit_frac=0.05),
    # four row groups, one per wave (R = 16 + 7*64 = 464; D = 64: R = 16 + 4*107 = 444)
    "four-row-groups": W("f11", B=1, Hq=14, Hkv=2, D=128, N=16900, W=64, C=16, budget=2048, n_centroids=16),
    "four-row-groups-d64": W("f12", B=1, Hq=8, Hkv=2, D=64, N=16461, W=107, C=16, budget=1900, n_centroids=8),
    # budgets above the selection's bin count: its kept tokens go out without the LDS staging
    "budget-above-bins": W("f13", B=1, Hq=8, Hkv=2, D=128, N=24000, W=16, C=8, budget=6000),
    "budget-above-bins-d64": W("f14", B=1, Hq=8, Hkv=2, D=64, N=20000, W=16, C=8, budget=3000),
}


def _evict_both(d, x, mean=False, causal=False):
    """bkv_evict on x and the chained entry points on a copy; returns both."""
    opt = dict(rope_cos=x["rope_cos"], rope_sin=x["rope_sin"], mean=mean, causal=causal)
    K2, V2 = x["K"].clone(), x["V"].clone()
    ws = bkv.workspace(d, bkv.OP_EVICT)
    kept = torch.full((d.B, d.Hkv, d.n_keep), -1, dtype=torch.int32, device="cuda")
    scores = torch.full((d.B, d.Hkv, d.N), float("nan"), device="cuda")
    bkv.evict(d, x["K"], x["V"], x["q_win"], x["beacons"], x["counts"], ws, kept=kept, scores=scores, **opt)
    assert bkv.device_status(ws) == bkv.OK
    ws2 = bkv.workspace(d, bkv.OP_EVICT)
    kept2 = torch.full_like(kept, -1)
    scores2 = torch.empty_like(scores)
    bkv.score(d, K2, x["q_win"], x["beacons"], x["counts"], scores2, ws2, **opt)
    bkv.topk(d, scores2, kept2)
    bkv.compact(d, K2, V2, kept2, ws2)
    assert bkv.device_status(ws2) == bkv.OK
    return (kept, scores), (kept2, scores2, K2, V2)


def _check(w, x0, d, mean=False, causal=False, seed_note=""):
    xd = {k: v.cuda() for k, v in x0.items()}
    (kept, scores), (kept2, scores2, K2, V2) = _evict_both(d, xd, mean, causal)
    s_gpu, k_gpu = host(scores).numpy(), host(kept).numpy()
    heads = None if w.P <= 16 else [(b, h) for b in (0, w.B - 1) for h in (0, w.Hkv - 1)]
    s_ref, _ = oracle.score(x0["K"], x0["q_win"], x0["beacons"], x0["counts"], N=w.N, rope_cos=x0["rope_cos"],
                            rope_sin=x0["rope_sin"], heads=heads, threads=8, agg="mean" if mean else "max",
                            causal=causal)
    sel = (slice(None),) if heads is None else tuple(np.array(heads).T)
    err = assert_scores_close(s_gpu[sel], s_ref[sel])
    # isolation checks on every head
    np.testing.assert_array_equal(oracle.topk(s_gpu.astype(np.float64), w.budget, w.W, w.n_prefix), k_gpu)
    Kr, Vr = oracle.compact(x0["K"], x0["V"], k_gpu)
    n = d.n_keep
    assert np.array_equal(raw_bits(xd["K"])[..., :n, :], Kr[..., :n, :].view(np.uint16)), "K differs"
    assert np.array_equal(raw_bits(xd["V"])[..., :n, :], Vr[..., :n, :].view(np.uint16)), "V differs"
    assert np.array_equal(raw_bits(xd["K"])[..., n:, :], raw_bits(x0["K"])[..., n:, :]), "rows past n moved"
    # the chained entry points agree bit for bit
    np.testing.assert_array_equal(host(scores2).numpy(), s_gpu)
    np.testing.assert_array_equal(host(kept2).numpy(), k_gpu)
    assert torch.equal(K2.view(torch.int16), xd["K"].view(torch.int16))
    assert torch.equal(V2.view(torch.int16), xd["V"].view(torch.int16))
    say(f"  {seed_note}max |score diff| {err:.2e}")


@pytest.mark.parametrize("name", list(CHAINED))
def test_evict_of_small_layers(name):
    w = CHAINED[name]
    big = w.P * w.N > 1 << 20
    x = synth.make_layer(w, seed=71, device="cuda" if big else "cpu")
    x = {k: host(v) for k, v in x.items()}
    d = dims_of(w)
    assert fuses(d) == (name == "many-heads")
    say(f"evict {name} {d}")
    _check(w, x, d)


@pytest.mark.parametrize("mean,causal", [(True, False), (False, True), (True, True)])
@pytest.mark.parametrize("name", ["prefix", "four-row-groups"])
def test_evict_of_small_layers_options(name, mean, causal):
    w = CHAINED[name]
    x = synth.make_layer(w, seed=72, device="cpu")
    d = dims_of(w)
    say(f"evict mean={mean} causal={causal} {d}")
    _check(w, x, d, mean, causal)


@pytest.mark.parametrize("distinct", [1, 3, 40])
def test_evict_of_small_layers_bulk_ties(distinct):
    # keys repeat `distinct` rows only: scores tie in bulk, so the threshold
    # value is shared by many candidates (one distinct row: every candidate
    # ties) and the kept ones among equals must be the lowest indices
    w = W("f10", B=2, Hq=8, Hkv=2, D=128, N=16500, W=16, C=4, budget=2100, n_prefix=2)
    x = synth.make_layer(w, seed=73, device="cpu")
    g = torch.Generator().manual_seed(74)
    pick = torch.randint(0, distinct, (w.B, w.Hkv, w.N), generator=g)
    K = x["K"]
    rows = K[:, :, :distinct].clone()
    K[:] = torch.gather(rows, 2, pick.unsqueeze(-1).expand(-1, -1, -1, w.D))
    d = dims_of(w)
    say(f"evict with {distinct} distinct keys {d}")
    _check(w, x, d, seed_note=f"{distinct} distinct: ")


# The fused launch takes layers of 1.05 or 1.5 million tokens or more (by their
# heads' length) that keep at most half of them.  About 100 heads of one query
# head each reach every part of it: ragged tails, the prefix, D = 64, budgets
# above the selection's bin count, chunks of unequal length, no window, no
# beacons, a longer allocation, the options, and bulk ties.
FUSED = {  # workload, mean, causal, tokens allocated past N
    "ragged-prefix": (W("g1", B=12, Hq=8, Hkv=8, D=128, N=16391, W=16, C=8, budget=2000, n_prefix=5), False, False, 0),
    "d64-causal": (W("g2", B=13, Hq=8, Hkv=8, D=64, N=15999, W=9, C=3, budget=2048), False, True, 0),
    "half-kept-mean": (W("g3", B=6, Hq=8, Hkv=8, D=128, N=32768, W=16, C=8, budget=16384), True, False, 0),
    "nine-tiles": (W("g4", B=12, Hq=32, Hkv=8, D=128, N=17003, W=32, C=16, budget=1000, revisit_frac=0.05), True, True, 0),
    "no-window": (W("g6", B=13, Hq=8, Hkv=8, D=64, N=15501, W=0, C=8, budget=1000), False, False, 37),
    "no-beacons": (W("g7", B=7, Hq=8, Hkv=8, D=128, N=20011, W=24, C=0, budget=3001, n_prefix=1), False, True, 5),
    "few-long-heads": (W("g8", B=11, Hq=6, Hkv=3, D=64, N=32767, W=7, C=64, budget=9000), False, False, 1),
}


def _fused_inputs(w, seed, extra=0):
    d = dims_of(w, N_cap=w.N + extra)
    assert fuses(d)
    x = synth.make_layer(w, seed=seed, device="cuda", N_cap=w.N + extra)
    return d, {k: host(v) for k, v in x.items()}


@pytest.mark.parametrize("name", list(FUSED))
def test_fused_launch_on_large_layers(name):
    w, mean, causal, extra = FUSED[name]
    d, x = _fused_inputs(w, 75, extra)
    say(f"fused launch {name} {d}")
    _check(w, x, d, mean, causal)


def test_fused_launch_with_outputs_in_the_workspace():
    # scores and kept left to the workspace: the same rows, bit for bit
    w = W("g9", B=12, Hq=8, Hkv=8, D=64, N=16397, W=16, C=8, budget=2000, n_prefix=3)
    d, x = _fused_inputs(w, 78)
    a, b = ({k: v.cuda() for k, v in x.items()} for _ in range(2))
    kept = torch.empty(d.B, d.Hkv, d.n_keep, dtype=torch.int32, device="cuda")
    scores = torch.empty(d.B, d.Hkv, d.N, device="cuda")
    say(f"fused launch, outputs in the workspace {d}")
    for y, out in ((a, {"kept": kept, "scores": scores}), (b, {})):
        ws = bkv.workspace(d, bkv.OP_EVICT)
        bkv.evict(d, y["K"], y["V"], y["q_win"], y["beacons"], y["counts"], ws, rope_cos=y["rope_cos"],
                  rope_sin=y["rope_sin"], **out)
        assert bkv.device_status(ws) == bkv.OK
    assert torch.equal(a["K"].view(torch.int16), b["K"].view(torch.int16))
    assert torch.equal(a["V"].view(torch.int16), b["V"].view(torch.int16))


@pytest.mark.parametrize("distinct", [1, 3, 40])
def test_fused_launch_bulk_ties(distinct):
    w = W("g5", B=12, Hq=8, Hkv=8, D=64, N=16500, W=16, C=4, budget=2100, n_prefix=2)
    d, x = _fused_inputs(w, 76)
    g = torch.Generator().manual_seed(77)
    pick = torch.randint(0, distinct, (w.B, w.Hkv, w.N), generator=g)
    x["K"] = torch.gather(x["K"][:, :, :distinct], 2, pick.unsqueeze(-1).expand(-1, -1, -1, w.D))
    say(f"fused launch with {distinct} distinct keys {d}")
    _check(w, x, d, seed_note=f"{distinct} distinct: ")
