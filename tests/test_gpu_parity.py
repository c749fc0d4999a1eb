"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element by element.

Bars: logits rel-L2 <= 1e-5 (fp32 accumulation of a fp32 dot product against the float64 oracle
rounded to fp32); integer tables bit-exact and combine weights |err| <= 1e-6 GIVEN IDENTICAL
LOGITS - where the library computes the logits itself, the oracle's routing is run on the
library's own logits, and the number of decisions that the float64-logit routing would take
differently (near-ties flipped by rounding) is printed, not asserted; layer output rel-L2 <= 1e-5
(fp32 workload) / <= 2e-2 (bf16 workloads), plus a per-row and a per-element bound (below), so that
a wrong store mask on a ragged tile cannot hide in the norm.
"""
import dataclasses
import re

import numpy as np
import pytest
import torch

import paper_2402_12399_amd as rr
from oracle import rectify_router as orc
from paper_2402_12399_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

MODES = [(), ("ir",), ("fr",), ("ir", "fr")]

# Output bounds.  bf16 layers round three times on the way to an output element - h, y and the
# output itself, each by at most 2^-9 of the value - and the rounding of h enters an element as a
# random-sign sum over d_ff terms, i.e. about 2^-9 of the row's rms.  Per element:
# |got - want| <= ELEM_ATOL * rms(want row) + ELEM_RTOL * |want| (16 such roundings + 2^-7 of the
# element); per row: |got - want|_2 <= ROW_RTOL * |want|_2.  fp32 layers accumulate in fp32:
# about sqrt(d_ff) * 2^-24 of the row's rms per element.  A masked-out or misplaced store is an
# error of the order of the row's rms itself.
OUT_BOUNDS = {"bf16": dict(l2=2e-2, row=2.0 ** -6, elem_atol=2.0 ** -5, elem_rtol=2.0 ** -7),
              "f32": dict(l2=1e-5, row=3e-5, elem_atol=5e-5, elem_rtol=1e-5)}


def _assert_output_close(got, want, dtype, what=""):
    """got, want: float64 [n, d] outputs of the same tokens."""
    b = OUT_BOUNDS[dtype]
    err = gu.rel_l2(got, want)
    assert err <= b["l2"], f"{what} rel-L2 {err}"
    wn = np.linalg.norm(want, axis=1)
    row_err = np.linalg.norm(got - want, axis=1)
    bad = row_err > b["row"] * np.maximum(wn, 1e-30)
    assert not bad.any(), f"{what} {int(bad.sum())} rows off, worst {float((row_err / np.maximum(wn, 1e-30)).max())}"
    rms = wn / np.sqrt(want.shape[1])
    tol = b["elem_atol"] * rms[:, None] + b["elem_rtol"] * np.abs(want)
    off = np.abs(got - want) > tol
    assert not off.any(), (f"{what} {int(off.sum())} elements off, first at {np.argwhere(off)[0].tolist()}: "
                           f"got {got[tuple(np.argwhere(off)[0])]} want {want[tuple(np.argwhere(off)[0])]}")
    return err


def _flipped_decisions(tables, ref):
    """How many entries of the integer tables the routing from the oracle's own float64 logits takes
    differently from the routing on the library's logits (reported, not asserted)."""
    return {n: int((np.asarray(tables[n]) != np.asarray(ref[n])).sum()) if np.shape(tables[n]) == np.shape(ref[n])
            else -1 for n in ("rank_expert", "slot", "ir_expert")}


def _oracle_tables(a, cfg, mode, arrival=False, quota=False):
    return orc.route(a, cfg.k, cfg.G, cfg.capacity_factor, "ir" in mode, "fr" in mode,
                     orc.POLICY_ARRIVAL if arrival else orc.POLICY_SCORE, quota)


# ------------------------------------------------------------------ routing tables, identical logits
DISPATCH_CASES = [
    # T, E, G, k, cf, ties
    (256, 8, 2, 1, 1.0, False),
    (1000, 8, 4, 2, 1.25, False),     # ragged last token block
    (1000, 6, 2, 2, 0.5, True),       # E not a power of two, many ties, +-0
    (4099, 16, 1, 1, 1.0, True),      # prime T, one group
    (3 * 128, 64, 8, 2, 0.75, False),
    (5000, 64, 8, 4, 2.0, True),      # largest k, k+1 rounds
    (130, 4, 2, 3, 3.0, False),       # k+1 == E
    (64, 2, 2, 2, 1.0, True),         # k == E: no Fill-in possible
    (20000, 32, 8, 1, 0.5, False),
]


@pytest.mark.parametrize("T,E,G,k,cf,ties", DISPATCH_CASES)
@pytest.mark.parametrize("mode", MODES, ids=["vanilla", "ir", "fr", "ir+fr"])
def test_dispatch_tables_bit_exact(T, E, G, k, cf, ties, mode):
    if "fr" in mode and k + 1 > E:
        pytest.skip("Fill-in needs k+1 <= E")
    a = wl.synthetic_logits(T, E, seed=T + E + k, bias_std=1.0, ties=ties)
    for arrival in (False, True):
        cfg = rr.RRConfig(T, 64, 0, E, k, G, cf, rr.RR_F32, rr.RR_ACT_SWIGLU, gu.flags_of(mode, arrival))
        got = gu.run_dispatch(cfg, a)
        gu.assert_tables_equal(got, _oracle_tables(a, cfg, mode, arrival))


def test_dispatch_extreme_cases():
    # every token wants the same expert; capacity 1; capacity >= T; all scores equal
    T, E = 700, 8
    a = np.zeros((T, E), dtype=np.float32)
    a[:, 3] = 5.0
    for cf, k in [(1.0, 1), (0.001, 2), (float(E), 2)]:
        cfg = rr.RRConfig(T, 64, 0, E, k, 2, cf, rr.RR_F32, rr.RR_ACT_SWIGLU, rr.RR_INTRA_GPU | rr.RR_FILL_IN)
        gu.assert_tables_equal(gu.run_dispatch(cfg, a), _oracle_tables(a, cfg, ("ir", "fr")))
    a[:] = 1.0
    cfg = rr.RRConfig(T, 64, 0, E, 2, 4, 1.0, rr.RR_F32, rr.RR_ACT_SWIGLU, rr.RR_INTRA_GPU | rr.RR_FILL_IN)
    gu.assert_tables_equal(gu.run_dispatch(cfg, a), _oracle_tables(a, cfg, ("ir", "fr")))
    # a single token
    a1 = wl.synthetic_logits(1, 4, seed=9)
    cfg = rr.RRConfig(1, 64, 0, 4, 2, 1, 1.0, rr.RR_F32, rr.RR_ACT_SWIGLU, rr.RR_INTRA_GPU | rr.RR_FILL_IN)
    gu.assert_tables_equal(gu.run_dispatch(cfg, a1), _oracle_tables(a1, cfg, ("ir", "fr")))


def test_dispatch_deterministic():
    a = wl.synthetic_logits(30000, 64, seed=77, ties=True)
    cfg = rr.RRConfig(30000, 64, 0, 64, 2, 8, 0.75, rr.RR_F32, rr.RR_ACT_SWIGLU, rr.RR_INTRA_GPU | rr.RR_FILL_IN)
    first = gu.run_dispatch(cfg, a)
    for _ in range(3):
        again = gu.run_dispatch(cfg, a)
        for name in gu.INT_TABLES + ("combine_w",):
            assert np.array_equal(first[name], again[name]), name


# The selection's histogram of score values: scores whose range is no fp32 number, that lie within a few ulps, that are denormal,
# spread over many powers of two (nearly all in one bin), or tied en masse; lists of one register trip, of several,
# and cut into short segments, with a capacity that keeps few and one that keeps most.
def _odd_scores(kind, T, E):
    rng = np.random.default_rng(T + E)
    if kind == "wide":
        return (rng.uniform(-1, 1, (T, E)) * 3.3e38).astype(np.float32)
    if kind == "ulps":
        return (1.0 + rng.integers(0, 40, (T, E)) * 2.0 ** -23).astype(np.float32)
    if kind == "denormal":
        return (rng.integers(-3000, 3000, (T, E)) * 1e-42).astype(np.float32)
    if kind == "geometric":
        return (rng.choice([-1.0, 1.0], (T, E)) * 2.0 ** rng.uniform(-120, 100, (T, E))).astype(np.float32)
    a = rng.standard_normal((T, E)).astype(np.float32)  # "ties": most scores one of five values
    return np.where(rng.random((T, E)) < 0.9, np.round(a), a).astype(np.float32)


@pytest.mark.parametrize("kind", ["wide", "ulps", "denormal", "geometric", "ties"])
@pytest.mark.parametrize("T,E,G,k,cf,quota", [
    (3000, 6, 1, 2, 0.5, False), (16385, 2, 1, 1, 0.9, False), (33000, 4, 2, 1, 0.05, False), (33000, 2, 1, 1, 0.3, False),
    (4 * 2560, 4, 4, 1, 0.7, True)])
def test_dispatch_odd_scores_bit_exact(kind, T, E, G, k, cf, quota):
    a = _odd_scores(kind, T, E)
    cfg = rr.RRConfig(T, 64, 0, E, k, G, cf, rr.RR_F32, rr.RR_ACT_SWIGLU, gu.flags_of(("ir", "fr"), False, quota))
    want = _oracle_tables(a, cfg, ("ir", "fr"), False, quota)
    want["combine_w"] = _weights_of(a, want, k)
    gu.assert_tables_equal(gu.run_dispatch(cfg, a), want)


def _weights_of(a, tables, k):
    """Eq. 2 / Eq. 3 weights of oracle tables with the softmax over the processed experts alone: the oracle's, ratios of
    exponentials over all experts, are 0 / 0 where scores lie hundreds apart."""
    rank, slot, ir = tables["rank_expert"], tables["slot"], tables["ir_expert"]
    s = np.full((len(a), k + 2), -np.inf)
    rows = np.arange(len(a))
    for r in range(k + 1):
        s[:, r] = np.where(slot[:, r] >= 0, a[rows, rank[:, r]].astype(np.float64), -np.inf)
    s[:, k + 1] = np.where(ir >= 0, a[rows, ir].astype(np.float64), -np.inf)
    count = np.ones_like(s)
    count[:, k + 1] = k - (slot[:, :k] >= 0).sum(axis=1)  # Eq. 3: the dropped choices
    top = s.max(axis=1, keepdims=True)
    e = np.where(np.isfinite(s), count * np.exp(s - np.where(np.isfinite(top), top, 0.0)), 0.0)
    return e / np.maximum(e.sum(axis=1, keepdims=True), 1e-300)


# Scores that crowd a histogram of equal bins: one far from all others, many far away, two clusters, a grid (one score in the
# bin, many times), a cluster of many scores in one bin; lists held by one workgroup, by segments, and of per-group capacity.
def _crowded_scores(kind, T, E):
    rng = np.random.default_rng(T + E)
    a = rng.standard_normal((T, E))
    if kind == "one high":
        a[T // 3] = 1e4 * np.arange(1, E + 1)
    if kind == "one low":
        a[T // 3] = -1e4 * np.arange(1, E + 1)
    if kind == "many far":
        a[::50] *= 1e6
    if kind == "two clusters":
        a += 1e6 * (rng.random((T, E)) < 0.5)
    if kind == "grid":
        a = np.round(a * 4) / 4
    if kind == "one bin":
        a = np.where(rng.random((T, E)) < 0.7, 1 + rng.integers(0, 8192, (T, E)) * 2.0 ** -20, 8 * rng.random((T, E)))
    return a.astype(np.float32)


@pytest.mark.parametrize("kind", ["one high", "one low", "many far", "two clusters", "grid", "one bin"])
@pytest.mark.parametrize("T,E,G,k,cf,quota", [
    (1500, 3, 1, 1, 0.4, False), (8190, 4, 1, 2, 0.5, False), (20001, 2, 1, 1, 0.6, False), (33000, 2, 1, 1, 0.2, False),
    (60000, 4, 2, 2, 0.3, False), (4 * 2560, 4, 4, 1, 0.5, True)])
def test_dispatch_crowded_scores_bit_exact(kind, T, E, G, k, cf, quota):
    a = _crowded_scores(kind, T, E)
    cfg = rr.RRConfig(T, 64, 0, E, k, G, cf, rr.RR_F32, rr.RR_ACT_SWIGLU, gu.flags_of(("ir", "fr"), False, quota))
    want = _oracle_tables(a, cfg, ("ir", "fr"), False, quota)
    want["combine_w"] = _weights_of(a, want, k)
    gu.assert_tables_equal(gu.run_dispatch(cfg, a), want)


# The threshold at the lowest key of a crowded bin, and one to either side: keys of the bin below share its leading digits.
@pytest.mark.parametrize("kept", [1943, 3133, 4307, 5427])
def test_dispatch_threshold_at_the_end_of_a_bin(kept):
    rng = np.random.default_rng(9)
    T = 6000
    s = np.where(rng.random(T) < 0.8, 1 + rng.integers(0, 8192, T) * 2.0 ** -20, 8 * rng.random(T))
    a = np.stack([s, np.full(T, -1.0)], axis=1).astype(np.float32)
    for m in (kept - 1, kept, kept + 1):
        cfg = rr.RRConfig(T, 64, 0, 2, 1, 1, (m - 0.5) * 2 / T, rr.RR_F32, rr.RR_ACT_SWIGLU, 0)
        assert rr.rr_slots_per_expert(cfg) == m
        gu.assert_tables_equal(gu.run_dispatch(cfg, a), _oracle_tables(a, cfg, ()))


# Intra-GPU counts per 1024 tokens: from 4096 experts x 128-token blocks on, up to 8192 experts x 1024-token blocks; ragged ends.
@pytest.mark.parametrize("T,E", [(8192, 64), (8196, 64), (9220, 60), (131072, 64), (131076, 64)])
def test_dispatch_intra_gpu_blocks_bit_exact(T, E):
    a = wl.synthetic_logits(T, E, seed=T % 1000, bias_std=1.0, ties=False)
    cfg = rr.RRConfig(T, 64, 0, E, 1, 4, 0.6, rr.RR_F32, rr.RR_ACT_SWIGLU, gu.flags_of(("ir",)))
    gu.assert_tables_equal(gu.run_dispatch(cfg, a), _oracle_tables(a, cfg, ("ir",)))


# Small batches whose candidates count the keys that beat theirs (up to 128 tokens, more than 32 lists), and their neighbours:
# every token on few experts, ties, arrival order, per-group capacity, one token.
@pytest.mark.parametrize("T,E,G,k,cf,arrival,quota", [
    (128, 16, 4, 2, 0.5, False, False), (129, 16, 4, 2, 0.5, False, False), (128, 11, 1, 2, 0.25, False, False),
    (128, 64, 8, 4, 1.0, False, False), (1, 64, 1, 4, 1.0, False, False), (100, 32, 2, 1, 0.3, True, False),
    (128, 34, 1, 2, 0.5, False, True)])
@pytest.mark.parametrize("ties", [False, True])
def test_dispatch_counted_candidates_bit_exact(T, E, G, k, cf, arrival, quota, ties):
    if T % G:
        G = 1
    a = wl.synthetic_logits(T, E, seed=T + E, bias_std=2.0, ties=ties)
    a[:, E // 2] += np.float32(4.0)  # one list with nearly every token
    cfg = rr.RRConfig(T, 64, 0, E, k, G, cf, rr.RR_F32, rr.RR_ACT_SWIGLU, gu.flags_of(("ir", "fr"), arrival, quota))
    gu.assert_tables_equal(gu.run_dispatch(cfg, a), _oracle_tables(a, cfg, ("ir", "fr"), arrival, quota))


LONG_LIST_CASES = [
    # T, E, G, k, cf, bias of expert 1, ties, arrival, quota
    (300000, 8, 2, 2, 0.5, 4.0, False, False, False),   # one expert draws ~all first choices: a list of ~290 K candidates, split
    (300032, 8, 2, 1, 1.0, 4.0, True, False, False),    # the same with scores tied en masse: the sample cannot separate them
    (200000, 4, 2, 2, 3.0, 3.0, False, False, False),   # long lists kept whole (capacity above the candidates)
    (262144, 8, 2, 2, 0.75, 4.0, False, True, False),   # long lists, arrival order
    (4 * 65536, 4, 4, 1, 0.4, 5.0, False, False, True), # per-group capacity: every group's piece of the array is long
    (500000, 64, 8, 2, 0.75, 2.0, False, False, False), # 64 experts, moderate skew: long and short lists side by side
]


@pytest.mark.parametrize("T,E,G,k,cf,hot,ties,arrival,quota", LONG_LIST_CASES)
def test_dispatch_long_lists_bit_exact(T, E, G, k, cf, hot, ties, arrival, quota):
    """Selection lists far longer than one workgroup's registers (a skewed router): tables bit-exact."""
    a = wl.synthetic_logits(T, E, seed=T % 1000 + E, bias_std=0.5, ties=ties)
    a[:, 1] += np.float32(hot)
    a[:, min(3, E - 1)] += np.float32(hot / 2)
    cfg = rr.RRConfig(T, 64, 0, E, k, G, cf, rr.RR_F32, rr.RR_ACT_SWIGLU, gu.flags_of(("ir", "fr"), arrival, quota))
    gu.assert_tables_equal(gu.run_dispatch(cfg, a), _oracle_tables(a, cfg, ("ir", "fr"), arrival, quota))


# Token orders that defeat a sample of 64 evenly spaced runs of 64 candidates: the highest scores all in those runs, or none; and
# runs of neighbours with nearly the same score.  Lists just under and over what one workgroup holds, and long ones.
@pytest.mark.parametrize("T,cf", [(20000, 0.5), (24576, 0.2), (24577, 0.2), (60000, 0.2)])
@pytest.mark.parametrize("kind", ["in the runs", "outside", "alike"])
def test_dispatch_misleading_token_order_bit_exact(T, cf, kind):
    rng = np.random.default_rng(T)
    s = rng.standard_normal(T)
    runs = (np.arange(64)[:, None] * (T // 64) + np.arange(64)).ravel()
    if kind == "in the runs":
        s[runs] += 8
    if kind == "outside":
        s[runs] -= 8
    if kind == "alike":
        s = np.repeat(rng.standard_normal(T // 64 + 1), 64)[:T] + 0.01 * s
    a = np.stack([s, np.full(T, -40.0)], axis=1).astype(np.float32)  # all tokens choose expert 0
    cfg = rr.RRConfig(T, 64, 0, 2, 1, 1, cf, rr.RR_F32, rr.RR_ACT_SWIGLU, gu.flags_of(("ir", "fr")))
    gu.assert_tables_equal(gu.run_dispatch(cfg, a), _oracle_tables(a, cfg, ("ir", "fr")))


# ------------------------------------------------------------------ router scores
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,d,E,k", [(256, 64, 8, 1), (1000, 264, 6, 2), (513, 1024, 64, 2), (2048, 2048, 16, 1)])
def test_router_scores(dtype, T, d, E, k):
    rng = np.random.default_rng(T + d)
    x = wl._store(rng.standard_normal((T, d), dtype=np.float32), dtype)
    wr = rng.standard_normal((E, d), dtype=np.float32) * np.float32(0.05)
    b = rng.standard_normal(E).astype(np.float32)
    cfg = rr.RRConfig(T, d, 0, E, k, 1, 1.0, rr.RR_F32 if dtype == "f32" else rr.RR_BF16)
    logits = torch.empty((T, E), dtype=torch.float32, device="cuda")
    probs = torch.empty((T, E), dtype=torch.float32, device="cuda")
    ranks = torch.empty((T, k + 1), dtype=torch.int32, device="cuda")
    for bias in (b, None):
        rr.rr_router_scores(cfg, gu.to_device(x, dtype), torch.from_numpy(wr).cuda(),
                            None if bias is None else torch.from_numpy(bias).cuda(), logits, probs, ranks)
        torch.cuda.synchronize()
        want = orc.router_scores(wl.values_f32(x, dtype), wr, bias)
        got = logits.cpu().numpy()
        assert gu.rel_l2(got.astype(np.float64), want.astype(np.float64)) <= 1e-5
        assert np.abs(got - want).max() <= 1e-5 * max(1.0, np.abs(want).max())
        # d p = p (d a - sum p d a): at most twice the logit error, plus fp32 rounding of exp and the sum
        assert np.abs(probs.cpu().numpy() - orc.softmax_probs(want)).max() <= 2e-5 * max(1.0, np.abs(want).max()) + 1e-6
        # ranking: equal to the oracle's wherever the oracle's scores are not within rounding of a tie
        want_rank = orc.rank_experts(want, k + 1)
        got_rank = ranks.cpu().numpy()
        srt = -np.sort(-want.astype(np.float64), axis=1)
        clear = (srt[:, :k + 1] - srt[:, 1:k + 2]).min(axis=1) > 1e-4 if E > k + 1 else np.ones(T, bool)
        assert np.array_equal(got_rank[clear], want_rank[clear])
        assert clear.mean() > 0.99


# The K-split router's numbers of waves: 16, 8 and 4, on both sides of one workgroup per CU (8192 tokens), for every
# number of column fragments; rows that are no multiple of a macro-step.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,d,E,k", [(8192, 2056, 33, 2), (8193, 2056, 33, 2), (8193, 1032, 17, 1), (8193, 1032, 5, 1), (300, 1032, 64, 3)])
def test_router_scores_waves(dtype, T, d, E, k):
    test_router_scores(dtype, T, d, E, k)


# ------------------------------------------------------------------ whole layer
def _forward_case(w, mode, inputs, sample=None, arrival=False, quota=False, logits_l2=1e-5):
    cfg = gu.config_of(w, mode, arrival, T=inputs["x"].shape[0], quota=quota)
    dev = {n: (torch.from_numpy(inputs[n]).cuda() if n in ("w_router", "bias") and inputs[n] is not None
               else gu.to_device(inputs[n], w.dtype)) for n in ("x", "w_router", "bias", "w1", "w3", "w2")}
    out, tables, logits = gu.run_forward(cfg, dev)
    f32 = lambda n: None if inputs[n] is None else wl.values_f32(inputs[n], w.dtype)
    policy = orc.POLICY_ARRIVAL if arrival else orc.POLICY_SCORE
    a = orc.router_scores(f32("x"), inputs["w_router"], inputs["bias"])
    assert gu.rel_l2(logits.astype(np.float64), a.astype(np.float64)) <= logits_l2
    # identical logits: the oracle routes the library's own logits
    want_tables = orc.route(logits, w.k, w.G, w.capacity_factor, "ir" in mode, "fr" in mode, policy, quota)
    gu.assert_tables_equal(tables, want_tables, cw_atol=1e-6)
    print("[parity] %s %s: decisions flipped by logit rounding: %s" % (
        w.name, "+".join(mode) or "vanilla",
        _flipped_decisions(want_tables, orc.route(a, w.k, w.G, w.capacity_factor, "ir" in mode, "fr" in mode, policy, quota))))
    want_out = orc.moe_output(f32("x"), want_tables, w.k, f32("w1"), f32("w3"), f32("w2"), w.act, tokens=sample)
    got = gu.to_host_f64(out)
    assert np.isfinite(got).all()  # every row is written, also those that no sample looks at
    if sample is not None:
        got = got[sample]
    err = _assert_output_close(got, want_out, w.dtype, w.name)
    unprocessed = np.flatnonzero(want_tables["combine_w"].sum(axis=1) == 0)
    assert (gu.to_host_f64(out)[unprocessed] == 0).all()
    return err


@pytest.mark.parametrize("mode", MODES, ids=["vanilla", "ir", "fr", "ir+fr"])
def test_forward_c1_fp32(mode):
    _forward_case(wl.C1, mode, wl.make_inputs(wl.C1))


def test_forward_c1_arrival_policy():
    _forward_case(wl.C1, ("ir", "fr"), wl.make_inputs(wl.C1), arrival=True)


SMALL_BF16 = [
    wl.Workload("s1", 1024, 256, 512, 8, 2, 2, 1.25, "bf16", "swiglu", "normal:0.5", 11),
    wl.Workload("s2", 1000, 136, 264, 6, 2, 1, 0.5, "bf16", "swiglu", "zipf:1.5", 12),   # ragged everything
    wl.Workload("s3", 768, 128, 256, 4, 4, 1, 1.0, "bf16", "gelu", "normal:1.0", 13),
    wl.Workload("s4", 600, 72, 200, 4, 2, 2, 1.0, "f32", "swiglu", "normal:1.0", 14),
    # the LDS-DMA GEMM at its shortest K (three chunks, both projections) with gathered rows
    wl.Workload("s5", 1536, 192, 192, 4, 2, 2, 1.0, "bf16", "swiglu", "normal:0.5", 15),
    # GELU variant of the LDS-DMA GEMM with the fused gather; d_ff not a multiple of the column tile
    wl.Workload("s6", 1024, 256, 384, 4, 2, 1, 1.0, "bf16", "gelu", "normal:1.0", 16),
    # more tiles than compute units at three chunks per tile (every workgroup streams from one tile
    # into the next); the down projection's only column tile is narrower than the tile
    wl.Workload("s7", 2048, 192, 5632, 4, 2, 1, 1.0, "bf16", "swiglu", "zipf:1.1", 17),
]


@pytest.mark.parametrize("w", SMALL_BF16, ids=[w.name for w in SMALL_BF16])
@pytest.mark.parametrize("mode", [(), ("ir", "fr")], ids=["vanilla", "ir+fr"])
def test_forward_small(w, mode):
    _forward_case(w, mode, wl.make_inputs(w))


def _full_size_case(w, mode, n_sample=1024, quota=False, report_flips=True):
    """Full-size workload in the configuration the benchmark times; oracle outputs on a token sample."""
    dev = wl.make_inputs_device(w)
    cfg = gu.config_of(w, mode, quota=quota)
    out, tables, logits = gu.run_forward(cfg, dev)
    x = wl.values_f32(gu.to_host_storage(dev["x"]), w.dtype)
    wr, b = dev["w_router"].cpu().numpy(), None if dev["bias"] is None else dev["bias"].cpu().numpy()
    a = orc.router_scores(x, wr, b)
    assert gu.rel_l2(logits.astype(np.float64), a.astype(np.float64)) <= 1e-5
    # identical logits: the oracle routes the library's own logits
    want = orc.route(logits, w.k, w.G, w.capacity_factor, "ir" in mode, "fr" in mode, quota=quota)
    gu.assert_tables_equal(tables, want, cw_atol=1e-6)
    if report_flips:
        print("[parity] %s %s: decisions flipped by logit rounding: %s" % (
            w.name, "+".join(mode) or "vanilla",
            _flipped_decisions(want, orc.route(a, w.k, w.G, w.capacity_factor, "ir" in mode, "fr" in mode, quota=quota))))
    sample = np.sort(np.random.default_rng(w.seed).choice(w.T, n_sample, replace=False))

    class PerExpert:  # expert weights are pulled to the host one expert at a time
        def __init__(self, t):
            self.t, self.shape = t, t.shape

        def __getitem__(self, j):
            return wl.values_f32(gu.to_host_storage(self.t[j]), w.dtype)

    want_out = orc.moe_output(x, want, w.k, PerExpert(dev["w1"]), PerExpert(dev["w3"]), PerExpert(dev["w2"]),
                              w.act, tokens=sample)
    assert bool(torch.isfinite(out).all())  # every row is written, also those that the sample leaves out
    got = gu.to_host_f64(out[torch.from_numpy(sample).cuda()])
    _assert_output_close(got, want_out, w.dtype, w.name)
    unprocessed = torch.from_numpy(np.flatnonzero(want["combine_w"].sum(axis=1) == 0)).cuda()
    assert (out[unprocessed] == 0).all()
    return tables


def test_forward_is_deterministic():
    """The layer has no atomics on data and a fixed reduction order: repeated calls on the same
    inputs must give the same bits (an LDS or load-ordering race in the grouped GEMM would not)."""
    w = wl.C2
    dev = wl.make_inputs_device(w)
    cfg = gu.config_of(w, ("ir", "fr"))
    first, _, _ = gu.run_forward(cfg, dev, want_tables=False)
    first = first.clone()
    for _ in range(4):
        again, _, _ = gu.run_forward(cfg, dev, want_tables=False)
        assert torch.equal(first.view(torch.int16), again.view(torch.int16))


def test_forward_with_internal_tables_and_logits():
    """tables and logits are optional outputs of rr_moe_forward: without them the call keeps both in
    its workspace and must produce the same bits."""
    w = SMALL_BF16[4]
    inputs = wl.make_inputs(w)
    cfg = gu.config_of(w, ("ir", "fr"))
    dev = {n: (torch.from_numpy(inputs[n]).cuda() if n in ("w_router", "bias") and inputs[n] is not None
               else gu.to_device(inputs[n], w.dtype)) for n in ("x", "w_router", "bias", "w1", "w3", "w2")}
    want, _, _ = gu.run_forward(cfg, dev)
    out = torch.zeros_like(want)
    ws = rr.alloc_workspace(cfg)
    rr.rr_moe_forward(cfg, dev["x"], dev["w_router"], dev["bias"], dev["w1"], dev["w3"], dev["w2"], out, None, None, ws)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), want.view(torch.int16))


def test_forward_under_graph_capture():
    """rr_moe_forward only enqueues kernels on the caller's stream (no allocation, no memset, no
    synchronisation), so a caller may capture it in a HIP graph: every replay must give the eager bits,
    also with eager calls and synchronisations in between."""
    w = SMALL_BF16[0]
    inputs = wl.make_inputs(w)
    cfg = gu.config_of(w, ("ir", "fr"))
    dev = {n: (torch.from_numpy(inputs[n]).cuda() if n in ("w_router", "bias") and inputs[n] is not None
               else gu.to_device(inputs[n], w.dtype)) for n in ("x", "w_router", "bias", "w1", "w3", "w2")}
    out = torch.empty((cfg.T, cfg.d_model), dtype=torch.bfloat16, device="cuda")
    logits = torch.empty((cfg.T, cfg.E), dtype=torch.float32, device="cuda")
    tb, ws = rr.alloc_tables(cfg), rr.alloc_workspace(cfg)

    def step():
        rr.rr_moe_forward(cfg, dev["x"], dev["w_router"], dev["bias"], dev["w1"], dev["w3"], dev["w2"], out, tb, logits, ws)

    rr.rr_init()  # per-device host-side set-up happens outside the capture
    step()
    torch.cuda.synchronize()
    want = out.clone()
    want_slot = tb.slot.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for _ in range(3):
        out.zero_()
        tb.slot.fill_(-7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), want.view(torch.int16))
        assert torch.equal(tb.slot, want_slot)
        step()
        torch.cuda.synchronize()


@pytest.mark.parametrize("mode", MODES, ids=["vanilla", "ir", "fr", "ir+fr"])
def test_forward_c2_full_size(mode):
    _full_size_case(wl.C2, mode)


def test_forward_c3_full_size():
    _full_size_case(wl.C3, ("ir", "fr"), n_sample=512)


def test_forward_c5_full_size():
    t = _full_size_case(wl.C5, ("ir", "fr"), n_sample=512)
    # the workload is meant to overflow heavily and leave experts vacant
    assert (t["slot"][:, 0] < 0).mean() > 0.30
    assert (t["fill_topk"] < wl.C5.T * 0.5 / wl.C5.E).sum() >= 4


# Points of the capacity-factor sweep at the paper's layer shape (Tables 3-5): low capacity with
# Intra-GPU only, high capacity with Fill-in only, one expert per GPU.
SWEEP_POINTS = [
    ("top1_cf0.5_ir", dict(k=1, capacity_factor=0.5), ("ir",)),
    ("top2_cf3.0_fr", dict(k=2, capacity_factor=3.0), ("fr",)),
    ("top1_cf1.0_ir_one_expert_per_gpu", dict(k=1, capacity_factor=1.0, G=8), ("ir",)),
]


@pytest.mark.parametrize("name,change,mode", SWEEP_POINTS, ids=[p[0] for p in SWEEP_POINTS])
def test_forward_capacity_sweep_points_c3_shape(name, change, mode):
    _full_size_case(dataclasses.replace(wl.C3, name="c3_" + name, **change), mode, n_sample=256)


def test_c4_routing_full_size():
    """1M tokens, 64 experts, top-2: logits on sampled rows, tables bit-exact from identical logits."""
    w = wl.C4
    dev = wl.make_inputs_device(w, with_experts=False)
    cfg = gu.config_of(w)
    logits = torch.empty((w.T, w.E), dtype=torch.float32, device="cuda")
    rr.rr_router_scores(cfg, dev["x"], dev["w_router"], None, logits)
    torch.cuda.synchronize()
    sample = np.sort(np.random.default_rng(4).choice(w.T, 4096, replace=False))
    want = orc.router_scores(dev["x"][torch.from_numpy(sample).cuda()].cpu().numpy(), dev["w_router"].cpu().numpy())
    got = logits[torch.from_numpy(sample).cuda()].cpu().numpy()
    assert gu.rel_l2(got.astype(np.float64), want.astype(np.float64)) <= 1e-5
    # routing tables: the oracle and the HIP path are given the same fp32 logits (drawn on the host)
    a = wl.synthetic_logits(w.T, w.E, seed=4, bias_std=0.0)
    a *= np.float32(0.64)  # std of w.x at d_model 1024 with N(0, 0.02) router weights
    gu.assert_tables_equal(gu.run_dispatch(cfg, a), orc.route(a, w.k, w.G, w.capacity_factor, True, True))


def test_c4_forward_routing_full_size():
    """The routing-only workload through rr_moe_forward with d_ff = 0, exactly as the benchmark runs it
    (fp32, 1M tokens, d_model 1024, 64 experts: the streaming router's unpredicated path with the
    ranking fused into its epilogue, then every routing kernel).  Logits on sampled rows against Eq. 1
    in float64; then the oracle routes the library's own logits: every integer table bit-exact,
    weights within 1e-6 (Sec. 3, 4.1, 4.2, Eq. 3)."""
    w = wl.C4
    dev = wl.make_inputs_device(w, with_experts=False)
    cfg = rr.RRConfig(w.T, w.d_model, 0, w.E, w.k, w.G, w.capacity_factor, rr.RR_F32, rr.RR_ACT_SWIGLU,
                      rr.RR_INTRA_GPU | rr.RR_FILL_IN)
    tb, logits = rr.alloc_tables(cfg), torch.empty((w.T, w.E), dtype=torch.float32, device="cuda")
    ws = rr.alloc_workspace(cfg)
    rr.rr_moe_forward(cfg, dev["x"], dev["w_router"], dev["bias"], None, None, None, None, tb, logits, ws)
    torch.cuda.synchronize()
    sample = np.sort(np.random.default_rng(44).choice(w.T, 4096, replace=False))
    sel = torch.from_numpy(sample).cuda()
    want = orc.router_scores(dev["x"][sel].cpu().numpy(), dev["w_router"].cpu().numpy())
    got = logits[sel].cpu().numpy()
    assert gu.rel_l2(got.astype(np.float64), want.astype(np.float64)) <= 1e-5
    assert np.abs(got - want).max() <= 1e-5 * max(1.0, np.abs(want).max())
    a = logits.cpu().numpy()
    gu.assert_tables_equal(tb.to_host(), orc.route(a, w.k, w.G, w.capacity_factor, True, True), cw_atol=1e-6)


@pytest.mark.parametrize("dtype,d,E,k,G", [("f32", 256, 64, 2, 8), ("bf16", 512, 32, 1, 8), ("bf16", 256, 32, 2, 4)])
def test_routing_only_forward_exact_path_real_inputs(dtype, d, E, k, G):
    """The streaming router (more than 16 K tokens) on whole-chunk shapes - fp32 with 64 experts, bf16
    with 32 - with N(0,1) tokens and N(0,0.02) router weights: logits against Eq. 1 in float64, tables
    from the library's own logits."""
    T = 66048 + 256 * G  # not a multiple of the router's 256-token workgroup
    T += 8 * G
    rng = np.random.default_rng(d + E)
    x = wl._store(rng.standard_normal((T, d), dtype=np.float32), dtype)
    wr = rng.standard_normal((E, d), dtype=np.float32) * np.float32(0.02)
    b = (rng.standard_normal(E) * 0.5).astype(np.float32)
    cfg = rr.RRConfig(T, d, 0, E, k, G, 0.75, rr.RR_F32 if dtype == "f32" else rr.RR_BF16, rr.RR_ACT_SWIGLU,
                      rr.RR_INTRA_GPU | rr.RR_FILL_IN)
    tb, logits = rr.alloc_tables(cfg), torch.empty((T, E), dtype=torch.float32, device="cuda")
    ws = rr.alloc_workspace(cfg)
    rr.rr_moe_forward(cfg, gu.to_device(x, dtype), torch.from_numpy(wr).cuda(), torch.from_numpy(b).cuda(),
                      None, None, None, None, tb, logits, ws)
    torch.cuda.synchronize()
    want = orc.router_scores(wl.values_f32(x, dtype), wr, b)
    a = logits.cpu().numpy()
    assert gu.rel_l2(a.astype(np.float64), want.astype(np.float64)) <= 1e-5
    assert np.abs(a - want).max() <= 1e-5 * max(1.0, np.abs(want).max())
    gu.assert_tables_equal(tb.to_host(), orc.route(a, k, G, 0.75, True, True), cw_atol=1e-6)


@pytest.mark.parametrize("dtype,d,E,k,G", [("f32", 128, 64, 2, 8), ("f32", 384, 64, 3, 4), ("bf16", 256, 32, 1, 8),
                                           ("bf16", 768, 32, 2, 2)])
def test_routing_only_forward_exact_path_dyadic(dtype, d, E, k, G):
    """The same kernel path with small dyadic inputs: every dot product is exact, so the logits must
    equal the oracle's bit for bit, ties are frequent, and the tables must match exactly."""
    T = 65536 + 24 * G
    rng = np.random.default_rng(7 * d + E + k)
    x = rng.integers(-3, 4, size=(T, d)).astype(np.float32) / np.float32(2.0)
    wr = rng.integers(-4, 5, size=(E, d)).astype(np.float32) / np.float32(8.0)
    b = rng.integers(-8, 9, size=E).astype(np.float32) / np.float32(4.0)
    cfg = rr.RRConfig(T, d, 0, E, k, G, 0.75, rr.RR_F32 if dtype == "f32" else rr.RR_BF16, rr.RR_ACT_SWIGLU,
                      rr.RR_INTRA_GPU | rr.RR_FILL_IN)
    xs = wl._store(x, dtype)
    tb, logits = rr.alloc_tables(cfg), torch.empty((T, E), dtype=torch.float32, device="cuda")
    ws = rr.alloc_workspace(cfg)
    rr.rr_moe_forward(cfg, gu.to_device(xs, dtype), torch.from_numpy(wr).cuda(), torch.from_numpy(b).cuda(),
                      None, None, None, None, tb, logits, ws)
    torch.cuda.synchronize()
    a = orc.router_scores(wl.values_f32(xs, dtype), wr, b)
    assert np.array_equal(logits.cpu().numpy(), a)
    gu.assert_tables_equal(tb.to_host(), orc.route(a, k, G, 0.75, True, True))


@pytest.mark.parametrize("dtype,E,k,G", [("f32", 64, 2, 8), ("bf16", 16, 1, 4), ("f32", 24, 4, 2), ("f32", 33, 2, 1),
                                         ("bf16", 17, 1, 1)])
def test_routing_only_forward_large_batch(dtype, E, k, G):
    """Large batches take the streaming router whose epilogue also ranks (d_ff = 0: routing only); here
    d_model is not a whole number of K chunks and the expert counts do not fill the staged rows.
    Inputs are small dyadic rationals, so every dot product is exact in fp32 and in bf16 parts: the logits
    must equal the oracle's bit for bit, ties are frequent, and the tables must match exactly."""
    T, d = 66112 + 16 * G, 72
    rng = np.random.default_rng(E + k)
    x = rng.integers(-3, 4, size=(T, d)).astype(np.float32) / np.float32(2.0)
    wr = rng.integers(-4, 5, size=(E, d)).astype(np.float32) / np.float32(8.0)
    b = rng.integers(-8, 9, size=E).astype(np.float32) / np.float32(4.0)
    cfg = rr.RRConfig(T, d, 0, E, k, G, 0.75, rr.RR_F32 if dtype == "f32" else rr.RR_BF16, rr.RR_ACT_SWIGLU,
                      rr.RR_INTRA_GPU | rr.RR_FILL_IN)
    xs = wl._store(x, dtype)
    tb, logits = rr.alloc_tables(cfg), torch.empty((T, E), dtype=torch.float32, device="cuda")
    ws = rr.alloc_workspace(cfg)
    rr.rr_moe_forward(cfg, gu.to_device(xs, dtype), torch.from_numpy(wr).cuda(), torch.from_numpy(b).cuda(),
                      None, None, None, None, tb, logits, ws)
    torch.cuda.synchronize()
    a = orc.router_scores(wl.values_f32(xs, dtype), wr, b)
    assert np.array_equal(logits.cpu().numpy(), a)
    gu.assert_tables_equal(tb.to_host(), orc.route(a, k, G, 0.75, True, True))
    # the stand-alone router entry point takes the same kernel (without the ranking epilogue)
    probs = torch.empty_like(logits)
    ranks = torch.empty((T, k + 1), dtype=torch.int32, device="cuda")
    rr.rr_router_scores(cfg, gu.to_device(xs, dtype), torch.from_numpy(wr).cuda(), torch.from_numpy(b).cuda(),
                        logits, probs, ranks)
    torch.cuda.synchronize()
    assert np.array_equal(logits.cpu().numpy(), a)
    assert np.array_equal(ranks.cpu().numpy(), orc.rank_experts(a, k + 1))
    assert np.abs(probs.cpu().numpy() - orc.softmax_probs(a)).max() <= 1e-6


@pytest.mark.parametrize("dtype,E,k,G,quota", [("bf16", 32, 1, 8, False), ("f32", 16, 2, 4, True), ("bf16", 24, 3, 2, False)])
def test_routing_only_forward_mid_batch(dtype, E, k, G, quota):
    """Just above 16 K tokens: the smallest batches of the streaming router (its grid does not fill the
    chip), a ragged last workgroup, per-group capacity.  Exact dyadic inputs: logits and tables must
    match bit for bit."""
    T, d = (20480 if quota else 20000 + 8 * G), 136
    rng = np.random.default_rng(3 * E + k)
    x = rng.integers(-3, 4, size=(T, d)).astype(np.float32) / np.float32(2.0)
    wr = rng.integers(-4, 5, size=(E, d)).astype(np.float32) / np.float32(8.0)
    b = rng.integers(-8, 9, size=E).astype(np.float32) / np.float32(4.0)
    cfg = rr.RRConfig(T, d, 0, E, k, G, 0.75, rr.RR_F32 if dtype == "f32" else rr.RR_BF16, rr.RR_ACT_SWIGLU,
                      gu.flags_of(("ir", "fr"), False, quota))
    xs = wl._store(x, dtype)
    tb, logits = rr.alloc_tables(cfg), torch.empty((T, E), dtype=torch.float32, device="cuda")
    ws = rr.alloc_workspace(cfg)
    rr.rr_moe_forward(cfg, gu.to_device(xs, dtype), torch.from_numpy(wr).cuda(), torch.from_numpy(b).cuda(),
                      None, None, None, None, tb, logits, ws)
    torch.cuda.synchronize()
    a = orc.router_scores(wl.values_f32(xs, dtype), wr, b)
    assert np.array_equal(logits.cpu().numpy(), a)
    gu.assert_tables_equal(tb.to_host(), orc.route(a, k, G, 0.75, True, True, quota=quota))
    # the stand-alone entry point takes the same kernel without the fused ranking
    probs = torch.empty_like(logits)
    ranks = torch.empty((T, k + 1), dtype=torch.int32, device="cuda")
    rr.rr_router_scores(cfg, gu.to_device(xs, dtype), torch.from_numpy(wr).cuda(), torch.from_numpy(b).cuda(),
                        logits, probs, ranks)
    torch.cuda.synchronize()
    assert np.array_equal(logits.cpu().numpy(), a)
    assert np.array_equal(ranks.cpu().numpy(), orc.rank_experts(a, k + 1))
    assert np.abs(probs.cpu().numpy() - orc.softmax_probs(a)).max() <= 1e-6


# ------------------------------------------------------------------ capacity per group (Sec. 3 capacity read per GPU)
QUOTA_CASES = [
    # T, E, G, k, cf, ties
    (256, 8, 2, 1, 1.0, False),        # one token block per group
    (1024, 8, 1, 2, 1.25, False),      # one group: the global reading
    (1536, 6, 3, 2, 0.5, True),        # E and G not powers of two, many ties
    (8 * 128, 64, 8, 2, 0.75, False),  # per-group capacity of 2 slots
    (8 * 640, 64, 8, 4, 2.0, True),    # largest k
    (2 * 384, 4, 2, 3, 3.0, False),    # k+1 == E
    (2 * 128, 2, 2, 2, 1.0, True),     # k == E
    (5 * 4096, 30, 5, 1, 0.5, False),
    (2 * 33792, 16, 2, 2, 1.0, True),
]


@pytest.mark.parametrize("T,E,G,k,cf,ties", QUOTA_CASES)
@pytest.mark.parametrize("mode", MODES, ids=["vanilla", "ir", "fr", "ir+fr"])
def test_quota_dispatch_tables_bit_exact(T, E, G, k, cf, ties, mode):
    if "fr" in mode and k + 1 > E:
        pytest.skip("Fill-in needs k+1 <= E")
    a = wl.synthetic_logits(T, E, seed=T + E + k + 1, bias_std=1.0, ties=ties)
    for arrival in (False, True):
        cfg = rr.RRConfig(T, 64, 0, E, k, G, cf, rr.RR_F32, rr.RR_ACT_SWIGLU, gu.flags_of(mode, arrival, quota=True))
        assert rr.rr_slots_per_expert(cfg) == G * orc.capacity(T // G, E, cf)
        got = gu.run_dispatch(cfg, a)
        gu.assert_tables_equal(got, _oracle_tables(a, cfg, mode, arrival, quota=True))


def test_quota_dispatch_extreme_cases():
    # every token wants the same expert; per-group capacity 1; per-group capacity >= T/G; all scores equal
    T, E, G = 1024, 8, 4
    a = np.zeros((T, E), dtype=np.float32)
    a[:, 3] = 5.0
    flags = gu.flags_of(("ir", "fr"), quota=True)
    for cf, k in [(1.0, 1), (0.001, 2), (float(E), 2)]:
        cfg = rr.RRConfig(T, 64, 0, E, k, G, cf, rr.RR_F32, rr.RR_ACT_SWIGLU, flags)
        gu.assert_tables_equal(gu.run_dispatch(cfg, a), _oracle_tables(a, cfg, ("ir", "fr"), quota=True))
    a[:] = 1.0
    cfg = rr.RRConfig(T, 64, 0, E, 2, G, 1.0, rr.RR_F32, rr.RR_ACT_SWIGLU, flags)
    gu.assert_tables_equal(gu.run_dispatch(cfg, a), _oracle_tables(a, cfg, ("ir", "fr"), quota=True))
    # candidate lists of one group longer than the selection keeps in registers
    Tb = 2 * 32768
    a = wl.synthetic_logits(Tb, 4, seed=22, ties=True)
    a[:, 1] += 6.0
    cfg = rr.RRConfig(Tb, 64, 0, 4, 2, 2, 1.0, rr.RR_F32, rr.RR_ACT_SWIGLU, flags)
    gu.assert_tables_equal(gu.run_dispatch(cfg, a), _oracle_tables(a, cfg, ("ir", "fr"), quota=True))
    a = wl.synthetic_logits(T, E, seed=21)
    # one group is starved of an expert that the other floods: the flooded group may not borrow the idle slots
    a[: T // 2, 0] += 8.0
    a[T // 2:, 0] -= 8.0
    cfg = rr.RRConfig(T, 64, 0, E, 1, 2, 1.0, rr.RR_F32, rr.RR_ACT_SWIGLU, flags)
    got = gu.run_dispatch(cfg, a)
    gu.assert_tables_equal(got, _oracle_tables(a, cfg, ("ir", "fr"), quota=True))
    Cq = orc.capacity(T // 2, E, 1.0)
    assert (got["slot_token"][0, :Cq] >= 0).all() and (got["slot_token"][0, :Cq] < T // 2).all()
    assert ((got["slot_token"][0, Cq:] >= T // 2) | (got["slot_token"][0, Cq:] < 0)).all()


def test_quota_c4_routing_full_size():
    w = wl.C4
    cfg = gu.config_of(w, quota=True)
    a = wl.synthetic_logits(w.T, w.E, seed=5, bias_std=0.3)
    gu.assert_tables_equal(gu.run_dispatch(cfg, a), orc.route(a, w.k, w.G, w.capacity_factor, True, True, quota=True))


@pytest.mark.parametrize("mode", MODES, ids=["vanilla", "ir", "fr", "ir+fr"])
def test_quota_forward_c1_fp32(mode):
    _forward_case(wl.C1, mode, wl.make_inputs(wl.C1), quota=True)


QUOTA_SMALL = [w for w in SMALL_BF16 if (w.T // w.G) * w.G == w.T and (w.T // w.G) % 128 == 0]
QUOTA_SMALL += [
    # bf16 rows that are no whole K chunks, E not a power of two
    wl.Workload("q1", 1024, 136, 264, 6, 2, 1, 0.5, "bf16", "swiglu", "zipf:1.5", 31),
    # fp32 tiles, top-2, three groups
    wl.Workload("q2", 1152, 72, 200, 6, 3, 2, 1.0, "f32", "swiglu", "normal:1.0", 32),
]


@pytest.mark.parametrize("w", QUOTA_SMALL, ids=[w.name for w in QUOTA_SMALL])
@pytest.mark.parametrize("mode", [(), ("ir", "fr")], ids=["vanilla", "ir+fr"])
def test_quota_forward_small(w, mode):
    _forward_case(w, mode, wl.make_inputs(w), quota=True)


@pytest.mark.parametrize("mode", [(), ("ir", "fr")], ids=["vanilla", "ir+fr"])
def test_quota_forward_c2_full_size(mode):
    _full_size_case(wl.C2, mode, quota=True)


def test_quota_forward_c5_full_size():
    _full_size_case(wl.C5, ("ir", "fr"), n_sample=512, quota=True)


# ------------------------------------------------------------------ seeded random configurations
def test_dispatch_random_configurations():
    """Sixty seeded draws over the whole argument space of the routing tables (sizes on both sides of
    the small-batch path's limit, E, G, k, capacity factor, rectification modes, drop policy, capacity
    scope, tie density): tables bit-exact."""
    rng = np.random.default_rng(2024)
    done = 0
    while done < 60:
        G = int(rng.choice([1, 2, 3, 4, 8]))
        E = G * int(rng.integers(1, 64 // G + 1))
        k = int(rng.integers(1, 5))
        if k > E:
            continue
        quota = bool(rng.integers(0, 2))
        if quota:
            T = G * 128 * int(rng.integers(1, 12))
        elif rng.integers(0, 4) == 0:  # above 16 K tokens the selection lists are materialised (scan, scatter)
            T = G * int(rng.integers(16384 // G + 1, 40000 // G))
        else:
            T = G * int(rng.integers(1, 1500))
        mode = MODES[int(rng.integers(0, 4))]
        if "fr" in mode and k + 1 > E:
            continue
        cf = float(rng.choice([0.05, 0.3, 0.5, 0.75, 1.0, 1.25, 2.0, 4.0]))
        arrival = bool(rng.integers(0, 2))
        ties = bool(rng.integers(0, 2))
        a = wl.synthetic_logits(T, E, seed=1000 + done, bias_std=float(rng.choice([0.0, 1.0, 3.0])), ties=ties)
        cfg = rr.RRConfig(T, 64, 0, E, k, G, cf, rr.RR_F32, rr.RR_ACT_SWIGLU, gu.flags_of(mode, arrival, quota))
        try:
            gu.assert_tables_equal(gu.run_dispatch(cfg, a), _oracle_tables(a, cfg, mode, arrival, quota))
        except AssertionError as err:
            raise AssertionError(f"T={T} E={E} G={G} k={k} cf={cf} mode={mode} arrival={arrival} quota={quota} "
                                 f"ties={ties}: {err}") from None
        done += 1


def test_routing_only_forward_random_configurations():
    """The same through rr_moe_forward with d_ff = 0 (the router's fused ranking instead of topk_rank; every
    fourth draw is a batch for the streaming router): inputs are small dyadic rationals, so the logits are
    exact and the tables must match bit for bit."""
    rng = np.random.default_rng(77)
    done = 0
    while done < 32:
        G = int(rng.choice([1, 2, 4, 8]))
        E = G * int(rng.integers(1, 64 // G + 1))
        k = int(rng.integers(1, 4))
        if k + 1 > E:
            continue
        quota = bool(rng.integers(0, 2))
        if done % 4 == 3:  # above 16 K tokens: the streaming router and materialised selection lists
            T = G * 128 * int(rng.integers(130 // G + 1, 400 // G + 2)) if quota else G * int(rng.integers(16385 // G + 1, 70000 // G))
        else:
            T = G * 128 * int(rng.integers(1, 10)) if quota else G * int(rng.integers(10, 1200))
        d = 8 * int(rng.integers(2, 40))
        dtype = "bf16" if rng.integers(0, 2) else "f32"
        x = rng.integers(-3, 4, size=(T, d)).astype(np.float32) / np.float32(2.0)
        wr = rng.integers(-4, 5, size=(E, d)).astype(np.float32) / np.float32(8.0)
        b = rng.integers(-8, 9, size=E).astype(np.float32) / np.float32(4.0)
        cf = float(rng.choice([0.3, 0.75, 1.0, 1.5]))
        cfg = rr.RRConfig(T, d, 0, E, k, G, cf, rr.RR_F32 if dtype == "f32" else rr.RR_BF16, rr.RR_ACT_SWIGLU,
                          gu.flags_of(("ir", "fr"), False, quota))
        xs = wl._store(x, dtype)
        tb, logits = rr.alloc_tables(cfg), torch.empty((T, E), dtype=torch.float32, device="cuda")
        ws = rr.alloc_workspace(cfg)
        rr.rr_moe_forward(cfg, gu.to_device(xs, dtype), torch.from_numpy(wr).cuda(), torch.from_numpy(b).cuda(),
                          None, None, None, None, tb, logits, ws)
        torch.cuda.synchronize()
        a = orc.router_scores(wl.values_f32(xs, dtype), wr, b)
        assert np.array_equal(logits.cpu().numpy(), a), (T, d, E, dtype)
        try:
            gu.assert_tables_equal(tb.to_host(), orc.route(a, k, G, cf, True, True, quota=quota))
        except AssertionError as err:
            raise AssertionError(f"T={T} d={d} E={E} G={G} k={k} cf={cf} {dtype} quota={quota}: {err}") from None
        done += 1


def test_forward_random_grouped_gemm_shapes():
    """Twelve seeded draws of bf16 layer shapes that take the LDS-DMA grouped GEMM (d_model and d_ff
    multiples of 64 from 192 up: ragged row tiles, column tiles narrower than the tile, few or many
    chunks per tile), over expert counts, k, modes, capacity scope and both activations.  Router
    inputs are small dyadic rationals, so logits and tables must match bit for bit."""
    rng = np.random.default_rng(5)
    done = 0
    while done < 12:
        G = int(rng.choice([1, 2, 4]))
        E = G * int(rng.integers(1, 16 // G + 1))
        k = int(rng.integers(1, 4))
        if k + 1 > E:
            continue
        quota = bool(rng.integers(0, 2))
        T = G * 128 * int(rng.integers(1, 17)) if quota else G * int(rng.integers(50, 2500))
        d = 64 * int(rng.integers(3, 17))
        F = 64 * int(rng.integers(3, 33))
        act = "swiglu" if rng.integers(0, 2) else "gelu"
        mode = MODES[int(rng.integers(0, 4))]
        cf = float(rng.choice([0.3, 0.75, 1.0, 1.5, 3.0]))
        x = rng.integers(-3, 4, size=(T, d)).astype(np.float32) / np.float32(2.0)
        wr = rng.integers(-4, 5, size=(E, d)).astype(np.float32) / np.float32(8.0)
        b = rng.integers(-8, 9, size=E).astype(np.float32) / np.float32(4.0)
        w1 = wl._store(rng.standard_normal((E, F, d), dtype=np.float32) * np.float32(0.05), "bf16")
        w3 = wl._store(rng.standard_normal((E, F, d), dtype=np.float32) * np.float32(0.05), "bf16") if act == "swiglu" else None
        w2 = wl._store(rng.standard_normal((E, d, F), dtype=np.float32) * np.float32(0.05), "bf16")
        xs = wl._store(x, "bf16")
        what = f"T={T} d={d} F={F} E={E} G={G} k={k} cf={cf} {act} mode={mode} quota={quota}"
        cfg = rr.RRConfig(T, d, F, E, k, G, cf, rr.RR_BF16, rr.RR_ACT_GELU if act == "gelu" else rr.RR_ACT_SWIGLU,
                          gu.flags_of(mode, False, quota))
        dev = {"x": gu.to_device(xs, "bf16"), "w_router": torch.from_numpy(wr).cuda(), "bias": torch.from_numpy(b).cuda(),
               "w1": gu.to_device(w1, "bf16"), "w3": gu.to_device(w3, "bf16"), "w2": gu.to_device(w2, "bf16")}
        out, tables, logits = gu.run_forward(cfg, dev)
        f32 = lambda s: None if s is None else wl.values_f32(s, "bf16")
        a = orc.router_scores(f32(xs), wr, b)
        assert np.array_equal(logits, a), what
        want = orc.route(a, k, G, cf, "ir" in mode, "fr" in mode, quota=quota)
        try:
            gu.assert_tables_equal(tables, want, cw_atol=1e-6)
            _assert_output_close(gu.to_host_f64(out), orc.moe_output(f32(xs), want, k, f32(w1), f32(w3), f32(w2), act),
                                 "bf16")
        except AssertionError as err:
            raise AssertionError(f"{what}: {err}") from None
        done += 1


# The grouped GEMM in small tiles: every shape of tile for either type, with ragged rows, columns and K (one chunk and
# less, a last chunk of one piece, exactly whole chunks), experts without rows, and both activations.
TILE_SHAPES = [
    # tile of the up / down projection, T, d_model, d_ff, E, G, k, dtype, act
    ("32x64 one row", 1, 64, 8, 4, 1, 1, "bf16", "swiglu"),
    ("32x64 K 8", 40, 8, 72, 4, 2, 2, "bf16", "gelu"),
    ("32x64 ragged", 70, 200, 136, 8, 2, 2, "bf16", "swiglu"),
    ("64x128 32x128", 900, 456, 1000, 6, 2, 2, "bf16", "gelu"),
    ("128x128 ragged K", 1300, 2056, 1032, 2, 1, 1, "bf16", "swiglu"),
    ("256x256 64x128", 1500, 264, 4104, 4, 1, 2, "bf16", "swiglu"),
    ("256x256 128x128", 2600, 584, 2056, 4, 2, 2, "bf16", "swiglu"),
    ("256x256 256x128 ragged K", 9001, 264, 2312, 4, 1, 2, "bf16", "gelu"),
    ("256x128 ragged K", 9001, 2312, 264, 4, 1, 1, "bf16", "swiglu"),
    ("256x256 ragged K", 3000, 2056, 776, 3, 1, 2, "bf16", "swiglu"),
    ("f32 32x64 one row", 1, 8, 40, 4, 1, 1, "f32", "gelu"),
    ("f32 32x64", 129, 800, 264, 4, 1, 2, "f32", "swiglu"),
    ("f32 32x128", 1900, 104, 1208, 4, 2, 2, "f32", "swiglu"),
    ("f32 64x128", 4032, 40, 3032, 2, 1, 1, "f32", "gelu"),
]


@pytest.mark.parametrize("case", TILE_SHAPES, ids=[c[0] for c in TILE_SHAPES])
def test_forward_tile_shapes(case):
    name, T, d, F, E, G, k, dtype, act = case
    w = wl.Workload(name, T, d, F, E, G, k, 1.0, dtype, act, "zipf:1.1", 40 + T % 97)
    shapes = gu.ffn_shapes(gu.config_of(w))
    for i, (bm, brows) in enumerate(re.findall(r"(\d+)x(\d+)", name)):  # the up projection's tiles, and the down projection's
        assert (shapes.bm[i], shapes.brows[i]) == (int(bm), int(brows))
    _forward_case(w, ("ir", "fr"), wl.make_inputs(w))


# fp32 in split tiles: ragged rows, columns and K (a last chunk of one piece; whole chunks), both tiles for both GEMMs, rows
# through slots, Intra-GPU lists and per-group rows.
SPLIT_SHAPES = [
    # tile of the up / down projection, T, d_model, d_ff, E, G, k, act, quota
    ("64x128 64x128", 4097, 520, 264, 3, 1, 2, "swiglu", False),
    ("64x128 128x128", 4097, 776, 264, 3, 1, 2, "swiglu", False),
    ("128x128 64x128", 4097, 520, 1032, 3, 1, 2, "gelu", False),
    ("128x128 128x128", 4097, 776, 392, 3, 1, 2, "swiglu", False),
    ("128x128 128x128", 4096, 800, 1032, 4, 4, 2, "gelu", True),
]


@pytest.mark.parametrize("case", SPLIT_SHAPES, ids=[f"{c[0]} {c[7]}{' quota' * c[8]}" for c in SPLIT_SHAPES])
def test_forward_split_tiles(case):
    name, T, d, F, E, G, k, act, quota = case
    w = wl.Workload(name, T, d, F, E, G, k, 1.0, "f32", act, "zipf:1.1", 40 + T % 97)
    shapes = gu.ffn_shapes(gu.config_of(w, quota=quota))
    assert [f"{m}x{n}" for m, n in zip(shapes.bm, shapes.brows)] == name.split()
    _forward_case(w, ("ir", "fr"), wl.make_inputs(w), quota=quota, sample=np.arange(0, T, 4))


@pytest.mark.parametrize("act", ["gelu", "swiglu"])
def test_forward_split_tiles_of_values_without_bf16_parts(act):
    """Weights that a bf16 part cannot hold (rounding to an infinity), infinities and NaN: what fp32 arithmetic makes of them,
    and nothing else in the layer's output moves.  (Small values: the two tests below.)"""
    T, d, F = 4097, 1032, 1032
    w = wl.Workload("special", T, d, F, 1, 1, 1, 1.0, "f32", act, "none", 92)
    assert list(gu.ffn_shapes(gu.config_of(w, ())).brows) == [128, 128]
    inp = wl.make_inputs(w)
    inp["x"][:, 5] *= np.float32(1e-38)          # times a weight of 3.4e38: an ordinary term
    inp["w1"][0, 40, 5] = inp["w1"][0, 700, 5] = np.float32(3.4e38)
    clean, clean_ref = _whole_layer(w, inp)
    assert np.linalg.norm(clean - clean_ref) <= 1e-5 * np.linalg.norm(clean_ref)
    inp["w2"][0, 300, 9] = np.inf                # output column 300: +-inf by the sign of inner unit 9, column 801: NaN
    inp["w2"][0, 801, 11] = np.nan
    got, ref = _whole_layer(w, inp)
    assert np.isinf(ref[:, 300]).mean() > 0.99   # (a unit that is zero makes NaN of an infinity)
    assert np.array_equal(np.where(np.isfinite(ref), 0, ref), np.where(np.isfinite(got), 0, got), equal_nan=True)
    others = np.setdiff1d(np.arange(d), [300, 801])
    assert np.linalg.norm(got[:, others] - ref[:, others]) <= 1e-5 * np.linalg.norm(ref[:, others])
    whole = np.array([c for c in others if c // 16 not in (300 // 16, 801 // 16)])  # a fragment is computed again as a whole
    assert np.array_equal(got[:, whole], clean[:, whole])


# fp32's whole range goes through the split tiles with all its bits: tokens and weights down to the smallest steps, and sums and
# operands beyond what the parts take (computed again).  x and the first weights are drawn at 2^ex and 2^ew, every fourth
# token at 2^(ex - 6): rows of one fragment differ.  Bounds per row: fp32 arithmetic on K = 1032 terms as elsewhere, 3e-5 of the row's norm,
# and half a step of 2^-149 for every term and result that is itself among the denormals: sqrt(1032) of them, far below the
# rows here (2^-126 at least, 2^-23 of it).
SPLIT_RANGES = [
    # act, ex, ew
    ("gelu", -116, 0), ("gelu", -118, 2), ("swiglu", -116, 80), ("swiglu", 76, -126), ("gelu", 84, -140), ("gelu", -138, 80),
    ("gelu", 20, 34), ("gelu", 95, -90), ("swiglu", -90, 100), ("swiglu", 0, 0),
]


@pytest.mark.parametrize("act,ex,ew", SPLIT_RANGES)
def test_forward_split_tiles_keep_the_range_of_fp32(act, ex, ew):
    T, d, F = 4097, 1032, 1032
    w = wl.Workload("range", T, d, F, 1, 1, 1, 1.0, "f32", act, "none", 93)
    assert list(gu.ffn_shapes(gu.config_of(w, ())).brows) == [128, 128]
    inp = wl.make_inputs(w)
    inp["x"] = np.ldexp(inp["x"], ex)
    inp["x"][::4] = np.ldexp(inp["x"][::4], -6)
    inp["w1"] = np.ldexp(inp["w1"], ew)
    if act == "swiglu":
        inp["w3"] = np.ldexp(inp["w3"], ew)
    got, ref = _whole_layer(w, inp)
    rows = np.linalg.norm(ref, axis=1)
    assert rows.min() > 2.0 ** -126 and np.isfinite(ref).all()
    err = np.linalg.norm(got - ref, axis=1) / rows
    assert err.max() <= 3e-5, (int(err.argmax()), float(err.max()))


@pytest.mark.parametrize("small,large", [(1e-38, 3e38), (1e-40, 3e38), (1e-38, 1e25)])
def test_forward_split_tiles_of_a_small_and_a_large_column(small, large):
    """One inner column of tiny activations (1e-40: denormal) against large weights: the terms that decide every inner unit."""
    T, d, F = 4097, 1032, 1032
    w = wl.Workload("column", T, d, F, 1, 1, 1, 1.0, "f32", "gelu", "none", 94)
    inp = wl.make_inputs(w)
    inp["x"] *= np.float32(small * large / 100.0)
    inp["x"][:, 77] = np.random.default_rng(5).standard_normal(T).astype(np.float32) * np.float32(small)
    inp["w1"][0, :, 77] = np.sign(inp["w1"][0, :, 77]) * np.float32(large)
    got, ref = _whole_layer(w, inp)
    x, w1 = inp["x"].astype(np.float64), inp["w1"][0, :64].astype(np.float64)
    assert np.linalg.norm(x[:, [77]] * w1[:, 77]) > 0.99 * np.linalg.norm(x @ w1.T)
    err = np.linalg.norm(got - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert err.max() <= 3e-5, float(err.max())


def _whole_layer(w, inp):
    """(output of a layer of one expert and room for every token, the same in float64)"""
    cfg, dev = gu.config_of(w, ()), {n: gu.to_device(v, "f32") for n, v in inp.items()}
    out = torch.full((w.T, w.d_model), float("nan"), device="cuda")
    rr.rr_moe_forward(cfg, dev["x"], dev["w_router"], dev["bias"], dev["w1"], dev["w3"], dev["w2"], out, None, None,
                      rr.alloc_workspace(cfg))
    x, w1, w2 = (torch.from_numpy(v).double() for v in (inp["x"], inp["w1"][0], inp["w2"][0]))
    g = x @ w1.T
    h = torch.nn.functional.gelu(g) if w.act == "gelu" else torch.nn.functional.silu(g) * (x @ torch.from_numpy(inp["w3"][0]).double().T)
    return out.cpu().numpy().astype(np.float64), (h @ w2.T).numpy()


def test_forward_more_tiles_than_a_grid_row():
    """2^24 tiles of the up projection: more workgroups than one grid dimension takes (128 GiB of inner activations)."""
    w = wl.Workload("many tiles", 1 << 20, 320, 32832, 1, 1, 1, 1.0, "f32", "swiglu", "none", 71)
    shapes = gu.ffn_shapes(gu.config_of(w, ()))
    assert shapes.bm[0] == 32 and (1 << 15) * (w.d_ff * 2 // shapes.brows[0]) * 256 > 1 << 32
    torch.cuda.empty_cache()
    _forward_case(w, (), wl.make_inputs(w), sample=np.random.default_rng(0).choice(w.T, 256, replace=False))
    torch.cuda.empty_cache()


# Rows and columns of 2^23 elements and more (64-bit addresses), both sides of the line, both types and activations, up
# projections that gather through slots, Intra-GPU lists and per-group rows.  fp32: K sums of 2^23 terms in 16 partial
# sums, each a chain of 2^17 MFMAs whose roundings add up to sqrt(2^17) * 2^-25 = 1.1e-5 of the sum, for the scores
# as well; two such sums make an inner unit (3e-5 of the row), and of 5e7 elements the worst is six deviations off.
@pytest.mark.parametrize("T,d,F,E,G,dtype,act,quota", [
    (6, 8, (1 << 23) - 8, 1, 1, "bf16", "swiglu", False), (6, 8, 1 << 23, 2, 1, "bf16", "swiglu", False),
    (40, 8, (1 << 23) + 8, 2, 2, "f32", "gelu", False), (6, (1 << 23) + 40, 8, 2, 1, "f32", "swiglu", False),
    (6, (1 << 23) + 40, 24, 1, 1, "bf16", "gelu", False), (128, 8, 1 << 23, 1, 1, "f32", "gelu", True)])
def test_forward_long_rows(monkeypatch, T, d, F, E, G, dtype, act, quota):
    monkeypatch.setitem(OUT_BOUNDS, "f32", dict(l2=3e-5, row=1e-4, elem_atol=2e-4, elem_rtol=1e-4))
    w = wl.Workload("long", T, d, F, E, G, 1, 0.5, dtype, act, "none", 80 + T)
    _forward_case(w, ("ir",), wl.make_inputs(w), quota=quota, sample=np.arange(0, T, 1 + T // 8), logits_l2=3e-5)


def _activation_of(g, act, d, F):
    """bf16 layer output act(g) for fp32 arguments g: one expert, g as the sum of its three bf16 parts (exact in fp32, so
    the pre-activation is g itself), an up projection of 1, and a down projection that passes one inner unit on."""
    g = torch.from_numpy(g)
    hi = g.bfloat16()
    lo = (g - hi.float()).bfloat16()
    x = torch.zeros(len(g), d, dtype=torch.bfloat16)
    x[:, 0], x[:, 1], x[:, 2] = hi, lo, (g - hi.float() - lo.float()).bfloat16()
    x[g.isinf(), :3] = 3e38  # finite tokens, an infinite sum (the other inner units have weights 0)
    x[:, 3] = 1
    w1 = torch.zeros(1, F, d, dtype=torch.bfloat16)
    w1[0, 0, :3] = 1
    w3 = torch.zeros_like(w1)
    w3[0, 0, 3] = 1
    w2 = torch.zeros(1, d, F, dtype=torch.bfloat16)
    w2[0, 0, 0] = 1
    cfg = rr.RRConfig(len(g), d, F, 1, 1, 1, 1.0, rr.RR_BF16, act, 0)
    out = torch.full((len(g), d), float("nan"), dtype=torch.bfloat16, device="cuda")
    rr.rr_moe_forward(cfg, x.cuda(), torch.zeros(1, d, device="cuda"), None, w1.cuda(),
                      w3.cuda() if act == rr.RR_ACT_SWIGLU else None, w2.cuda(), out, None, None, rr.alloc_workspace(cfg))
    torch.cuda.synchronize()
    return out[:, 0].float().cpu()


# Small tiles and the 256 x 256 kernel.  An fp32 value with relative error r (rms) rounds to the wrong bf16 neighbour with
# probability 2 r sqrt(2 / pi) / 2^-7.5 or so: for r = 4e-8 - half an ulp of the last operation and the erf's - 12 of 2^20
# arguments; twice that is allowed.  (Where 1 + erf cancels, g < -3, the error of g Phi(g) is absolute: not counted.)
@pytest.mark.parametrize("d,F", [(8, 8), (256, 256)])
@pytest.mark.parametrize("sigma", [0.3, 1.0])
def test_gelu_rounds_like_the_exact_function(d, F, sigma):
    g = (np.random.default_rng(3).standard_normal(1 << 20) * sigma).astype(np.float32)
    phi = 0.5 * torch.erfc(torch.from_numpy(g).double() * -(0.5 ** 0.5))
    want = (torch.from_numpy(g).double() * phi).bfloat16().float()
    wrong = (_activation_of(g, rr.RR_ACT_GELU, d, F) != want) & torch.from_numpy(g > -3)
    assert int(wrong.sum()) <= (24 if sigma < 1 else 36), int(wrong.sum())  # (negative arguments past -1 carry the cancellation)


# SwiGLU divides where K is ragged or shorter than three chunks: its tail stays down to the smallest normal numbers, where a
# reciprocal of 1 + exp(-g) is flushed to zero (g < -87.4).  __expf(-g): the exponent's rounding, 88 * 2^-24 relative.
@pytest.mark.parametrize("T,d,F", [(256, 8, 8), (256, 72, 64), (65536, 264, 256)])  # the last: 256 x 256 tiles
def test_swiglu_tail_of_ragged_layers(T, d, F):
    g = np.linspace(-88.0, -80.0, T).astype(np.float32)
    want = (torch.from_numpy(g).double() * torch.special.expit(torch.from_numpy(g).double()))
    got = _activation_of(g, rr.RR_ACT_SWIGLU, d, F).double()
    assert (got / want - 1).abs().max() <= 2.0 ** -8  # bf16 rounding


@pytest.mark.parametrize("d,F", [(8, 8), (256, 256)])
def test_gelu_of_large_and_infinite_arguments(d, F):
    g = torch.tensor([1e30, 3e38, 100.0, 13.0] * 40).bfloat16().float().numpy()
    assert torch.equal(_activation_of(g, rr.RR_ACT_GELU, d, F), torch.from_numpy(g).bfloat16().float())
    g[3::7] = np.inf
    got = _activation_of(g, rr.RR_ACT_GELU, d, F)
    assert torch.equal(got[3::7], torch.full_like(got[3::7], float("inf")))  # not NaN


# One expert: all tokens are its rows (no (k+1)-th choice, so no Fill-in), at sizes just under and over a tile's height.
@pytest.mark.parametrize("T,d,F,dtype,act", [(220, 256, 392, "bf16", "swiglu"), (257, 264, 384, "bf16", "gelu"),
                                             (56, 96, 200, "f32", "swiglu"), (65, 72, 264, "f32", "gelu")])
def test_forward_one_expert(T, d, F, dtype, act):
    for cf in (1.0, 0.4):  # everybody kept; most re-routed to the same expert
        w = wl.Workload("one expert", T, d, F, 1, 1, 1, cf, dtype, act, "none", 60 + T)
        _forward_case(w, ("ir",), wl.make_inputs(w))


# Top-1 with Intra-GPU Rectification and without Fill-in: every token has exactly one row, which the down projection stores, and
# nothing is combined.  Every tile that a down projection has, rows through slots, Intra-GPU lists and per-group rows, tables
# by one workgroup and by launches, ragged sizes; much and little dropped.
ONE_ROW_LAYERS = [
    # tile of the down projection, T, d_model, d_ff, E, G, cf, dtype, act, quota
    ("64x128 f32", 8194, 520, 264, 2, 1, 0.5, "f32", "swiglu", False), ("128x128 f32", 6001, 1032, 264, 2, 1, 1.0, "f32", "swiglu", False),
    ("32x64 f32", 130, 800, 264, 4, 2, 0.5, "f32", "swiglu", False), ("128x128 f32", 5632, 1032, 264, 4, 4, 0.5, "f32", "gelu", True),
    ("32x64 bf16", 40, 72, 136, 4, 2, 0.25, "bf16", "gelu", False), ("32x128 bf16", 700, 776, 264, 4, 1, 0.5, "bf16", "swiglu", False),
    ("64x128 bf16", 4097, 264, 264, 2, 1, 0.5, "bf16", "swiglu", False), ("128x128 bf16", 6001, 264, 264, 2, 1, 1.0, "bf16", "swiglu", False),
    ("256x128 bf16", 4097, 1032, 264, 2, 1, 0.5, "bf16", "swiglu", False), ("256x256 bf16", 7815, 2288, 888, 3, 1, 0.5, "bf16", "swiglu", False),
    ("256x256 bf16", 4096, 2040, 1512, 8, 2, 1.0, "bf16", "swiglu", True),
]


@pytest.mark.parametrize("case", ONE_ROW_LAYERS, ids=[f"{c[0]} T={c[1]}{' quota' * c[9]}" for c in ONE_ROW_LAYERS])
def test_forward_one_row_per_token(case):
    name, T, d, F, E, G, cf, dtype, act, quota = case
    w = wl.Workload(name, T, d, F, E, G, 1, cf, dtype, act, "zipf:1.1", 50 + T % 97)
    shapes = gu.ffn_shapes(gu.config_of(w, ("ir",), quota=quota))
    assert f"{shapes.bm[1]}x{shapes.brows[1]} {dtype}" == name
    rr.rr_profile_enable(True)
    try:
        _forward_case(w, ("ir",), wl.make_inputs(w), quota=quota)
        assert rr.rr_profile_read()["combine"][0] == 0
    finally:
        rr.rr_profile_enable(False)


# Batches whose tables one workgroup builds, and their borders: one token, a wave and one more or less, the most tokens
# (and one more), lists of one candidate and of all tokens, ranks shared by 1, 2, 4 and 8 lanes, every source of the ranking
# (logits; the router's partial scores or its own ranking in the forward call).
ONE_WORKGROUP = [
    # T, E, G, k, cf, quota
    (1, 2, 1, 1, 1.0, False),
    (63, 9, 1, 1, 0.5, False),
    (64, 64, 8, 2, 0.75, False),
    (65, 5, 1, 4, 1.0, False),
    (130, 64, 2, 4, 0.3, False),
    (256, 8, 2, 1, 40.0, False),     # queues far longer than the batch
    (512, 32, 4, 2, 1.0, True),
    (513, 24, 1, 3, 1.25, False),
    (1023, 16, 1, 2, 0.05, False),
    (1024, 3, 1, 2, 1.0, False),     # whole-batch lists, nothing placed in the last round
    (1024, 64, 8, 4, 0.5, True),
    (1025, 6, 1, 2, 1.0, False),
]


@pytest.mark.parametrize("T,E,G,k,cf,quota", ONE_WORKGROUP)
def test_small_batch_tables(T, E, G, k, cf, quota):
    for arrival in (False, True):
        for ties in (False, True):
            a = wl.synthetic_logits(T, E, seed=T + E, bias_std=1.5, ties=ties)
            cfg = rr.RRConfig(T, 64, 0, E, k, G, cf, rr.RR_F32, rr.RR_ACT_SWIGLU,
                              gu.flags_of(("ir", "fr"), arrival, quota))
            gu.assert_tables_equal(gu.run_dispatch(cfg, a), _oracle_tables(a, cfg, ("ir", "fr"), arrival, quota))
    rng = np.random.default_rng(T + 7 * E)
    for d in (72, 4160):  # one part of K, and as many as it is split into
        x = (rng.integers(-8, 9, (T, d)) / 8.0).astype(np.float32)  # dyadic: the scores are exact in any order
        wr = (rng.integers(-8, 9, (E, d)) / 16.0).astype(np.float32)
        cfg = rr.RRConfig(T, d, 0, E, k, G, cf, rr.RR_BF16, rr.RR_ACT_SWIGLU, gu.flags_of(("ir", "fr"), False, quota))
        tables, logits, ws = rr.alloc_tables(cfg), torch.empty((T, E), device="cuda"), rr.alloc_workspace(cfg)
        rr.rr_moe_forward(cfg, torch.from_numpy(x).cuda().bfloat16(), torch.from_numpy(wr).cuda(), None, None, None, None,
                          None, tables, logits, ws)
        torch.cuda.synchronize()
        a = logits.cpu().numpy()
        assert np.array_equal(a, (x.astype(np.float64) @ wr.astype(np.float64).T).astype(np.float32))
        gu.assert_tables_equal(tables.to_host(), _oracle_tables(a, cfg, ("ir", "fr"), False, quota))


# The line between one workgroup for all tables and the chain of launches: a batch on either side of it, for the terms it
# is made of (lists, candidates, Intra-GPU lists, capacity blocks), from logits, from the router's ranks and from its partial scores.
ONE_OR_CHAIN = [
    # T, E, G, k, mode, quota, d (0: from logits), one workgroup
    (480, 16, 1, 4, (), False, 0, True), (495, 16, 1, 4, (), False, 0, False),
    (660, 16, 1, 3, ("ir", "fr"), False, 0, True), (680, 16, 1, 3, ("ir", "fr"), False, 0, False),
    (1024, 32, 2, 2, ("ir", "fr"), True, 0, True), (1024, 64, 8, 4, ("ir", "fr"), True, 0, False),
    (960, 16, 1, 2, ("ir", "fr"), False, 1024, True), (976, 16, 1, 2, ("ir", "fr"), False, 1024, False),
    (128, 64, 1, 4, (), False, 2048, True), (400, 5, 1, 4, ("fr",), False, 64, True), (1000, 8, 1, 4, ("fr",), False, 2048, False),
]


@pytest.mark.parametrize("T,E,G,k,mode,quota,d,one", ONE_OR_CHAIN)
def test_tables_in_one_workgroup_or_by_launches(T, E, G, k, mode, quota, d, one):
    cfg = rr.RRConfig(T, d or 64, 0, E, k, G, 0.75, rr.RR_BF16, rr.RR_ACT_SWIGLU, gu.flags_of(mode, False, quota))
    tables, ws = rr.alloc_tables(cfg), rr.alloc_workspace(cfg)
    rr.rr_profile_enable(True)
    try:
        if d:
            rng = np.random.default_rng(T + d)
            x = (rng.integers(-8, 9, (T, d)) / 8.0).astype(np.float32)  # dyadic: the scores are exact in any order
            wr = (rng.integers(-8, 9, (E, d)) / 16.0).astype(np.float32)
            logits = torch.empty((T, E), device="cuda")
            rr.rr_moe_forward(cfg, torch.from_numpy(x).cuda().bfloat16(), torch.from_numpy(wr).cuda(), None, None, None,
                              None, None, tables, logits, ws)
            a = (x.astype(np.float64) @ wr.astype(np.float64).T).astype(np.float32)
            assert np.array_equal(logits.cpu().numpy(), a)
        else:
            a = wl.synthetic_logits(T, E, seed=T, bias_std=1.0, ties=True)
            rr.rr_rectified_dispatch(cfg, torch.from_numpy(a).cuda(), tables, ws)
        assert (rr.rr_profile_read()["route_small"][0] == 1) == one
    finally:
        rr.rr_profile_enable(False)
    gu.assert_tables_equal(tables.to_host(), _oracle_tables(a, cfg, mode, False, quota))


# The 256 x 256 kernel's last round: its tiles are cut by rows into as many parts as leave no CU idle.  First choices
# only, capacity T / E: the experts' rows, and so the cut of the up projection, follow from the tables.
CUT_TILES = [
    # T, d_model, d_ff, E, parts of a tile of the last round
    (4030, 232, 1336, 8, 2),  # no whole round before it; an expert without rows, and parts that are empty (27 rows)
    (5003, 232, 1048, 3, 3),  # the same; an expert of 5 rows
    (3500, 232, 4000, 5, 2),
    (3917, 232, 3352, 6, 3),  # experts of 7 and 10 rows
    (3500, 232, 3352, 5, 6),
    (3500, 232, 2992, 5, 8),
]


@pytest.mark.parametrize("T,d,F,E,parts", CUT_TILES)
def test_forward_cut_row_tiles(T, d, F, E, parts):
    w = wl.Workload(f"cut {parts}", T, d, F, E, 1, 1, 1.0, "bf16", "swiglu", "normal:0.5", 40 + T % 97)
    inputs = wl.make_inputs(w)
    first = orc.router_scores(wl.values_f32(inputs["x"], "bf16"), inputs["w_router"], inputs["bias"]).argmax(axis=1)
    rows = np.minimum(np.bincount(first, minlength=E), -(-T // E))
    left = int((-(-rows // 256)).sum()) * -(-F // 128) % 256
    assert min(256 // left, 8) == parts
    shapes = gu.ffn_shapes(gu.config_of(w, ()))
    assert (shapes.bm[0], shapes.brows[0]) == (256, 256)
    _forward_case(w, (), inputs)


# The same with the down projection in 256 x 256 tiles (256 output columns, the second store of single rows), the GELU up
# projection (256 columns), and rows through the per-group table.
CUT_DOWN_TILES = [
    # T, d_model, d_ff, E, G, act, quota, parts of a tile of the up / down projection's last round (1: not cut)
    (7815, 2288, 888, 3, 1, "swiglu", False, (1, 8)),
    (4096, 2040, 1512, 8, 2, "swiglu", True, (1, 2)),
    (4035, 2024, 1872, 8, 1, "gelu", False, (2, 2)),
    (4096, 1912, 1832, 8, 2, "gelu", True, (2, 2)),
]


@pytest.mark.parametrize("T,d,F,E,G,act,quota,parts", CUT_DOWN_TILES)
def test_forward_cut_row_tiles_of_the_down_projection(T, d, F, E, G, act, quota, parts):
    w = wl.Workload("cut down", T, d, F, E, G, 1, 1.0, "bf16", act, "normal:0.5", 40 + T % 97)
    inputs = wl.make_inputs(w)
    first = orc.router_scores(wl.values_f32(inputs["x"], "bf16"), inputs["w_router"], inputs["bias"]).argmax(axis=1)
    groups = first.reshape(G if quota else 1, -1)
    rows = sum(np.minimum(np.bincount(g, minlength=E), -(-groups.shape[1] // E)) for g in groups)
    row_tiles = int((-(-rows // 256)).sum())
    left = [row_tiles * -(-n // cols) % 256 for n, cols in ((F, 128 if act == "swiglu" else 256), (d, 256))]
    assert tuple(min(256 // n, 8) if n else 1 for n in left) == parts
    shapes = gu.ffn_shapes(gu.config_of(w, (), quota=quota))
    assert list(shapes.bm) == [256, 256] and list(shapes.brows) == [256, 256]
    _forward_case(w, (), inputs, quota=quota, sample=np.sort(np.random.default_rng(1).choice(T, 1024, replace=False)))


# x of 2 GiB and more: the dispatch gather is a pass of its own (32-bit buffer offsets), from slots and Intra-GPU lists and,
# with quotas, from the per-group rows.
@pytest.mark.parametrize("T,E,F,dtype,mode,quota", [(1 << 19, 4, 64, "f32", ("ir", "fr"), False), (1 << 20, 8, 192, "bf16", ("fr",), True)])
def test_forward_separate_gather(T, E, F, dtype, mode, quota):
    w = wl.Workload("gather", T, 1024, F, E, 2, 1, 1.0, dtype, "swiglu", "normal:0.5", 91)
    rr.rr_profile_enable(True)
    try:
        _full_size_case(w, mode, n_sample=256, quota=quota, report_flips=False)
        assert rr.rr_profile_read()["dispatch_gather"][0] == 1
    finally:
        rr.rr_profile_enable(False)


# Lists that their workgroup finds by itself, up to 16384 tokens: every number of tokens per thread (4, 8, 12, 16) with a
# last quadruple that is whole or ragged, the most rounds, and the first size past the limit.  The keys that the digit
# select meets: spread over the whole range of their type, all equal, and equal but for the last bits.
DIRECT_LISTS = [
    # T, E, k, cf, arrival, scores
    (1025, 2, 1, 0.5, False, "wide"), (4096, 6, 2, 0.75, False, "normal"), (4099, 8, 4, 0.6, True, "ties"),
    (8190, 8, 4, 0.5, False, "close"), (12289, 16, 2, 0.5, False, "wide"), (16384, 4, 2, 0.5, False, "normal"),
    (16383, 5, 3, 0.4, False, "equal"), (16385, 8, 2, 0.5, False, "close"), (5, 64, 2, 7000.0, False, "normal"),
]


@pytest.mark.parametrize("T,E,k,cf,arrival,scores", DIRECT_LISTS)
def test_dispatch_lists_found_by_their_workgroup(T, E, k, cf, arrival, scores):
    a = wl.synthetic_logits(T, E, seed=T + E, ties=scores == "ties")
    if scores == "wide":
        a = (np.sign(a) * np.exp2(4 * np.abs(a) - 12)).astype(np.float32)
    if scores == "equal":
        a[:] = -0.25
    if scores == "close":
        a = (1.0 + np.float32(2.0 ** -20) * np.round(a)).astype(np.float32)
    cfg = rr.RRConfig(T, 64, 0, E, k, 1, cf, rr.RR_F32, rr.RR_ACT_SWIGLU, gu.flags_of(("ir", "fr"), arrival))
    gu.assert_tables_equal(gu.run_dispatch(cfg, a), _oracle_tables(a, cfg, ("ir", "fr"), arrival, False))
