"""GPU parity of the HIP outer step against the CPU oracle (needs an MI355X).

Small cases span several 256-thread blocks and ragged tails; full-size
cases run units of each workload at their real shapes, through a handle
configured with every unit of the workload and stepped by
edit_outer_step_round, i.e. the launch configuration the benchmark times.
"""

import numpy as np
import pytest
import torch

from parity import NearTie, ParityRun, steady_ema
from paper_2412_07210_amd import EditOuter, EditOuterError, OuterConfig
from paper_2412_07210_amd import synth

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _run(run: ParityRun, rounds, verbose=True, **kw):
    try:
        recs = []
        for t in rounds:
            recs.append(run.round(t, verbose=verbose, **kw))
        return recs
    except NearTie as e:
        pytest.skip(str(e))
    finally:
        run.close()


def _expected_ema(wl, u, round_):
    """A settled EMA state (same on both sides) for unit u, to start a case
    after the warm-up without paying for the warm-up rounds."""
    return steady_ema(wl, wl.unit_numel(u), round_)


def _settle(h, wl, round_):
    """Give every unit of handle h the settled EMA state at `round_`."""
    for u in range(wl.num_units):
        h.state_set(u, *_expected_ema(wl, u, round_))


def _clean_pass(rec, K, bad=()):
    """The z-test ran and every worker outside `bad` passed it."""
    assert rec["z_tested"], "round not z-tested"
    clean = [j for j in range(K) if j not in bad]
    assert not rec["anomalous"][clean].any(), f"clean workers flagged: {list(rec['anomalous'])}"


# ------------------------------------------- one 1024x1024 linear layer, K = 4


def test_linear1m_k4_all_rounds():
    """1024x1024 fp32, K = 4: ten clean rounds, then worker 3 x50 is masked."""
    wl = synth.get("linear1m-k4")
    run = ParityRun(wl, [0], DEV)
    recs = _run(run, range(11), via_round=True)
    assert [int(x) for x in recs[10][0]["anomalous"]] == [0, 0, 0, 1]
    assert all(not r[0]["anomalous"].any() for r in recs[:10])
    assert recs[10][0]["clip_coef"] == 1.0


# ----------------------------------------------------- small and ragged


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("K", [1, 2, 3, 5, 8, 9, 11, 13, 16, 17, 24, 32])
def test_ragged_sizes(K, dtype):
    """Unit sizes around the 16-byte vector and the 256-thread block, K = 1..32
    (above 16 the Gram pass runs 21 to 36 matrix-core tiles): four rounds
    after the warm-up from a settled EMA state, the last with the last worker
    x40.  On the large units the clean workers pass the z-test and the x40
    one fails it."""
    sizes = [0, 1, 7, 8, 9, 255, 2049, 100_003, 1_000_005]
    wl = synth.small("llama1b-k8-bf16", sizes, num_workers=K, replica_dtype=dtype, clip_threshold=0.05,
                     name=f"ragged{K}{dtype}")
    W = wl.warmup_rounds
    run = ParityRun(wl, range(len(sizes)), DEV, ema_state={u: _expected_ema(wl, u, W) for u in range(len(sizes))})
    try:
        for t in range(W, W + 4):
            last = t == W + 3
            std = wl.worker_std(t) * (np.where(np.arange(K) == K - 1, 40.0, 1.0) if last else 1.0)
            recs = run.round(t, std=std, verbose=False)
            for n, r in zip(sizes, recs):
                if n >= 100_003:
                    _clean_pass(r, K, bad=(K - 1,) if last else ())
                    if last:
                        assert r["anomalous"][K - 1] == 1
    except NearTie as e:
        pytest.skip(str(e))
    finally:
        run.close()


@pytest.mark.parametrize("flags", range(8))
def test_flag_combinations(flags):
    """Every on/off combination of anomaly elimination, weighting and clipping
    (flags = 0 is the DiLoCo outer step)."""
    wl = synth.small("llama1b-k8-bf16", [300_001, 4096], num_workers=4, clip_threshold=0.2, name="flags")
    W = wl.warmup_rounds
    run = ParityRun(wl, [0, 1], DEV, flags=flags, ema_state={u: _expected_ema(wl, u, W) for u in (0, 1)})
    K = wl.num_workers
    try:
        for t in range(W, W + 4):
            std = wl.worker_std(t)
            if t == W + 3:
                std[1] *= 50
            recs = run.round(t, std=std, verbose=False)
            if flags & 1:  # anomaly elimination on: only the x50 worker is flagged
                _clean_pass(recs[0], K, bad=(1,) if t == W + 3 else ())
                assert recs[0]["anomalous"][1] == (t == W + 3)
    except NearTie as e:
        pytest.skip(str(e))
    finally:
        run.close()


def test_rollback_when_all_workers_flagged():
    """Every worker x100 after the warm-up: theta and b keep their values,
    all replicas get theta_t back (Sec. 3.2, Algorithm 2)."""
    wl = synth.small("llama1b-k8-bf16", [65_536 + 3], num_workers=4, name="rollback")
    W = wl.warmup_rounds
    run = ParityRun(wl, [0], DEV, ema_state={0: _expected_ema(wl, 0, W)})
    try:
        for t in range(W, W + 2):
            _clean_pass(run.round(t)[0], wl.num_workers)
        c = run.cases[0]
        theta_before = c.theta_h.copy()
        mom_before = c.mom_h.copy()
        recs = run.round(W + 2, std=wl.worker_std(W + 2) * 100)
        assert recs[0]["rolled_back"] == 1
        assert np.array_equal(c.theta_d.cpu().numpy(), theta_before)
        assert np.array_equal(c.mom_d.cpu().numpy(), mom_before)
        st = recs[0]["state"]
        assert st.rolled_back and st.anomalous.all() and st.clip_coef == 0.0
    finally:
        run.close()


def test_nonfinite_worker_is_masked():
    """A NaN in one replica makes its norm non-finite: that worker is masked
    (even during the warm-up) and the others still synchronize."""
    wl = synth.small("llama1b-k8-bf16", [10_000, 77], num_workers=5, name="nan")
    run = ParityRun(wl, [0, 1], DEV)
    try:
        recs = run.round(0, poison={2: (13, float("nan"))})
        for r in recs:
            assert list(r["anomalous"]) == [0, 0, 1, 0, 0]
            assert np.isfinite(run.cases[0].theta_d.cpu().numpy()).all()
        run.round(1, poison={0: (5, float("inf"))})
    finally:
        run.close()


# ------------------------------------------------------------ full size


def test_llama350m_f32_full_units():
    """Llama-350M-shaped units (12,847,104 fp32 elements, K = 8)."""
    wl = synth.get("llama350m-k8-f32")
    units = [0, 23]
    run = ParityRun(wl, units, DEV, ema_state={u: _expected_ema(wl, u, 10) for u in units})
    _run(run, [10, 11], via_round=True)


def test_llama350m_f32_every_unit_of_a_round():
    """All 24 units of the 350M workload in one full-size round, every element
    of theta, b and the replicas against the oracle."""
    wl = synth.get("llama350m-k8-f32")
    units = list(range(wl.num_units))
    run = ParityRun(wl, units, DEV, ema_state={u: _expected_ema(wl, u, 10) for u in units})
    _run(run, [10], verbose=False, via_round=True)


@pytest.mark.parametrize("entry", ["round", "layer"])
def test_llama1b_bf16_full_units_with_anomaly(entry):
    """Llama-1B-shaped units (51,384,320 elements, bf16 replicas, K = 8),
    rounds 18-19: round 19 has one worker x20, which must be masked.  Stepped
    as one round (both units in one batch) and unit by unit."""
    wl = synth.get("llama1b-k8-bf16")
    units = [0, 11]
    run = ParityRun(wl, units, DEV, ema_state={u: _expected_ema(wl, u, 18) for u in units})
    recs = _run(run, [18, 19], via_round=entry == "round")
    bad = list(wl.anomalies(19).keys())[0]
    for r in recs[1]:
        assert r["anomalous"][bad] == 1


def test_paper1b_full_units_with_anomaly():
    """The paper's own 1B shape (28,314,624 elements per layer, bf16, K = 8),
    first and last of its 32 units, round 19 with one worker x20."""
    wl = synth.get("paper1b-k8-bf16")
    assert wl.unit_numel(0) == 28_314_624 and wl.num_units == 32
    units = [0, 31]
    run = ParityRun(wl, units, DEV, ema_state={u: _expected_ema(wl, u, 19) for u in units})
    recs = _run(run, [19], via_round=True)
    bad = list(wl.anomalies(19).keys())[0]
    for r in recs[0]:
        assert r["anomalous"][bad] == 1 and r["anomalous"].sum() == 1


def test_llama7b_half_full_unit_clip_active():
    """7B half shard (101,191,680 elements, bf16, K = 8) with phi = 0.889: clipping active."""
    wl = synth.get("llama7b-half-k8-bf16")
    run = ParityRun(wl, [5], DEV, ema_state={5: _expected_ema(wl, 5, 10)})
    recs = _run(run, [10], via_round=True)
    assert recs[0][0]["clip_coef"] < 1.0


def test_aedit1b_k16_full_layer():
    """A-EDiT round on 1B shapes, K = 16: one layer's matrix unit (51,380,224)
    and its two 2,048-element RMSNorm units, three workers x30.  As one round:
    the gains are stepped whole in a launch of their own behind the matrix
    unit."""
    wl = synth.get("aedit1b-k16-bf16")
    units = [0, 1, 2]
    run = ParityRun(wl, units, DEV, ema_state={u: _expected_ema(wl, u, 10) for u in units})
    recs = _run(run, [10], via_round=True)
    flagged = sorted(wl.anomalies(10).keys())
    for r in recs[0]:
        assert sorted(np.flatnonzero(r["anomalous"]).tolist()) == flagged


# ------------------------------------------------- determinism, resume


def _fresh_inputs(wl, u, t, dev):
    th = wl.init_theta(u, dev)
    reps = [torch.empty(th.numel(), dtype=wl.torch_dtype, device=dev) for _ in range(wl.num_workers)]
    wl.fill_replicas(th, reps, u, t)
    return th, torch.zeros_like(th), reps


def test_bitwise_deterministic():
    wl = synth.small("llama1b-k8-bf16", [3_000_017], name="det")
    outs = []
    for _ in range(2):
        h = EditOuter(OuterConfig(wl.num_workers, wl.layer_numel, "bf16"), DEV)
        th, b, reps = _fresh_inputs(wl, 0, 0, DEV)
        h.step_layer(0, th, b, reps)
        torch.cuda.synchronize()
        outs.append((th.clone(), b.clone(), [r.clone() for r in reps], h.state_get(0)))
        h.close()
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    assert all(torch.equal(a, b) for a, b in zip(outs[0][2], outs[1][2]))
    assert np.array_equal(outs[0][3].norm, outs[1][3].norm)


def test_resume_from_saved_state_is_bitwise():
    """20 rounds straight equal 10 rounds, save EMA state, new handle, restore,
    10 rounds.  Both start from a settled state at the end of the warm-up, so
    the z-test runs (and passes) in every round."""
    wl = synth.small("llama1b-k8-bf16", [200_003], name="resume")
    W = wl.warmup_rounds
    cfg = OuterConfig(wl.num_workers, wl.layer_numel, "bf16", ema_warmup_rounds=W)

    def play(h, th, b, reps, rounds):
        for t in rounds:
            wl.fill_replicas(th, reps, 0, t)
            h.step_layer(0, th, b, reps)
        torch.cuda.synchronize()

    th, b, reps = _fresh_inputs(wl, 0, 0, DEV)
    th2, b2, reps2 = th.clone(), b.clone(), [r.clone() for r in reps]
    a = EditOuter(cfg, DEV)
    _settle(a, wl, W)
    play(a, th, b, reps, range(W, W + 20))
    s1 = EditOuter(cfg, DEV)
    _settle(s1, wl, W)
    play(s1, th2, b2, reps2, range(W, W + 10))
    st = s1.state_get(0)
    s1.close()
    s2 = EditOuter(cfg, DEV)
    s2.state_set(0, st.ema_mean, st.ema_std, st.round)
    play(s2, th2, b2, reps2, range(W + 10, W + 20))
    assert torch.equal(th, th2) and torch.equal(b, b2)
    sa, sb = a.state_get(0), s2.state_get(0)
    # the recipe's round-29 x20 worker is flagged and no other
    assert sa.round == sb.round == W + 20 and sa.z_tested
    assert sorted(np.flatnonzero(sa.anomalous).tolist()) == sorted(wl.anomalies(W + 19))
    assert np.array_equal(sa.ema_mean, sb.ema_mean) and np.array_equal(sa.ema_std, sb.ema_std)
    a.close()
    s2.close()


@pytest.mark.parametrize("K,dtype", [(8, "bf16"), (4, "f32"), (16, "bf16"), (32, "bf16")])
def test_round_and_streams_match_unit_by_unit(K, dtype):
    """A round (units in batches, small ones whole in launches of their own)
    and a 3-stream pipeline give the same bits as unit-by-unit calls, over
    several rounds (EMA state carried), units of mixed sizes and a unit order
    that is not the index order."""
    sizes = [1_000_000, 2048, 7, 3_000_017, 0, 65_536 + 3]
    wl = synth.small("llama1b-k8-bf16", sizes, num_workers=K, replica_dtype=dtype, name=f"round{K}{dtype}")
    W = wl.warmup_rounds
    order = [2, 0, 5, 1, 4, 3]
    results = []
    for mode in ("layer", "round", "streams"):
        h = EditOuter(OuterConfig(K, wl.layer_numel, dtype, ema_warmup_rounds=W), DEV)
        _settle(h, wl, W)
        units = [_fresh_inputs(wl, u, 0, DEV) for u in range(wl.num_units)]
        for t in range(W, W + 3):
            for u in range(wl.num_units):
                wl.fill_replicas(units[u][0], units[u][2], u, t)
            torch.cuda.synchronize()
            ordered = [units[u] for u in order]
            if mode == "layer":
                for u in order:
                    h.step_layer(u, *units[u])
            elif mode == "round":
                h.step_round(ordered, layers=order)
            else:
                h.step_round(ordered, layers=order, streams=[torch.cuda.Stream() for _ in range(3)])
            torch.cuda.synchronize()
        states = [h.state_get(u) for u in range(wl.num_units)]
        results.append((units, states))
        h.close()
    (ua, sa) = results[0]
    for (ub, sb) in results[1:]:
        for a, b in zip(ua, ub):
            assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
            assert all(torch.equal(x, y) for x, y in zip(a[2], b[2]))
        for x, y in zip(sa, sb):
            assert np.array_equal(x.norm, y.norm) and np.array_equal(x.ema_mean, y.ema_mean)
            assert x.round == y.round == W + 3
    assert sa[3].z_tested and not sa[3].anomalous.any()  # the 3M-element unit: every worker passes


# Units whose Gram pass is one block (at most 256 vectors: 2,048 bf16 or
# 1,024 fp32 elements) are stepped whole by a block each, gathered over the
# round into launches of up to 16 (8 above K = 16).  The sizes put six of them
# first, one and two between large units, and five at the end; bf16 K = 24 and
# fp32 K = 32 fill a launch before the round ends.
_SINGLE_BLOCK_SIZES = {
    "bf16": [0, 1, 7, 8, 2048, 2049, 300_001, 9, 65_537, 255, 2041, 1_000_003, 5, 2047, 16, 3, 2048],
    "f32": [0, 1, 7, 8, 1024, 1027, 300_001, 9, 65_537, 255, 1021, 1_000_003, 5, 1023, 16, 3, 1024],
}


@pytest.mark.parametrize("K,dtype", [(1, "bf16"), (3, "f32"), (8, "bf16"), (8, "f32"), (9, "bf16"),
                                     (16, "bf16"), (16, "f32"), (24, "bf16"), (32, "f32")])
def test_single_block_units_in_a_round_match_the_oracle(K, dtype):
    """A round dense in single-block units, stepped by edit_outer_step_round,
    against the oracle, from a settled EMA state: a clean round, a x40
    worker, every worker x1000 (all flagged: rollback), a NaN replica."""
    sizes = _SINGLE_BLOCK_SIZES[dtype]
    ve = 8 if dtype == "bf16" else 4
    wl = synth.small("llama1b-k8-bf16", sizes, num_workers=K, replica_dtype=dtype, clip_threshold=0.05,
                     name=f"single{K}{dtype}")
    W = wl.warmup_rounds
    run = ParityRun(wl, range(len(sizes)), DEV, ema_state={u: _expected_ema(wl, u, W) for u in range(len(sizes))})
    order = [int(i) for i in np.random.default_rng(K).permutation(len(sizes))] if K == 8 else None
    try:
        for t in range(W, W + 6):
            std = wl.worker_std(t)
            if t == W + 3:
                std = std * np.where(np.arange(K) == K - 1, 40.0, 1.0)
            if t == W + 4:
                std = std * 1000.0
            poison = {0: (0, float("nan"))} if t == W + 5 else None
            recs = run.round(t, std=std, poison=poison, via_round=True, order=order)
            big = [r for n, r in zip(sizes, recs) if n >= 65_537]
            if t < W + 3:  # clean rounds: the largest units flag no worker
                for r in big:
                    _clean_pass(r, K)
            if t == W + 4:  # the rollback path ran in some single-block unit
                assert any(r["rolled_back"] for n, r in zip(sizes, recs) if 64 <= n <= 256 * ve)
    except NearTie as e:
        pytest.skip(str(e))
    finally:
        run.close()


@pytest.mark.parametrize("K,dtype", [(2, "bf16"), (8, "bf16"), (8, "f32"), (16, "bf16"), (32, "bf16")])
def test_single_block_units_in_a_round_match_unit_by_unit(K, dtype):
    """The same round, its single-block units in launches of their own, gives
    the bits of unit-by-unit edit_outer_step_layer calls, over three rounds
    after the warm-up."""
    sizes = _SINGLE_BLOCK_SIZES[dtype]
    wl = synth.small("llama1b-k8-bf16", sizes, num_workers=K, replica_dtype=dtype, name=f"singlebits{K}{dtype}")
    W = wl.warmup_rounds
    order = [int(i) for i in np.random.default_rng(7).permutation(len(sizes))]
    results = []
    for mode in ("layer", "round"):
        h = EditOuter(OuterConfig(K, wl.layer_numel, dtype, ema_warmup_rounds=W), DEV)
        _settle(h, wl, W)
        units = [_fresh_inputs(wl, u, 0, DEV) for u in range(wl.num_units)]
        for t in range(W, W + 3):
            for u in range(wl.num_units):
                wl.fill_replicas(units[u][0], units[u][2], u, t)
            torch.cuda.synchronize()
            if mode == "layer":
                for u in order:
                    h.step_layer(u, *units[u])
            else:
                h.step_round([units[u] for u in order], layers=order)
            torch.cuda.synchronize()
        results.append((units, [h.state_get(u) for u in range(wl.num_units)]))
        h.close()
    (ua, sa), (ub, sb) = results
    for u, (a, b) in enumerate(zip(ua, ub)):
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]), f"unit {u}"
        assert all(torch.equal(x, y) for x, y in zip(a[2], b[2])), f"unit {u}"
    for x, y in zip(sa, sb):
        for f in ("norm", "ema_mean", "ema_std", "weight", "anomalous"):
            assert np.array_equal(getattr(x, f), getattr(y, f)), f
        assert x.synced_norm == y.synced_norm and x.clip_coef == y.clip_coef
        assert x.round == y.round == W + 3


# Round schedules (K <= 8): B = a unit of more than one Gram-pass block, which
# shares a batch's launches, S = a single-block unit, which is stepped whole
# in a launch of such units.  (name, sizes, timing)
_PAIR_SCHEDULES = [
    # B B B B B: one batch
    ("pairs", [300_001, 65_537, 1_000_003, 40_000, 123_457], 0),
    # eleven B: one longer batch
    ("pair_chain", [90_001, 65_537, 40_000, 70_007, 33_333, 100_000, 55_555, 81_920, 47_111, 60_000, 99_999], 0),
    # B B S B B B S S B: one batch, the three S after it
    ("pairs_riders", [300_001, 65_537, 2_048, 100_000, 77_777, 50_000, 1_000, 5, 150_001], 0),
    # B B S: a batch and a single S
    ("pair_rider_end", [300_001, 65_537, 33], 0),
    # nine B with every fourth unit timed: batches of three between timed units
    ("timed4", [200_003, 65_537, 90_000, 120_001, 40_000, 77_777, 100_000, 50_001, 70_000], 4),
    # eight B with every third unit timed: batches of two between timed units
    ("timed3", [200_003, 65_537, 90_000, 120_001, 40_000, 77_777, 100_000, 50_001], 3),
]


@pytest.mark.parametrize("K,dtype", [(8, "bf16"), (5, "f32")])
@pytest.mark.parametrize("name,sizes,every", _PAIR_SCHEDULES, ids=[s[0] for s in _PAIR_SCHEDULES])
def test_shared_gram_launches_match_unit_by_unit(K, dtype, name, sizes, every):
    """Rounds whose consecutive units share a Gram-pass launch, in the
    schedules the round path builds around it, give the bits of unit-by-unit
    edit_outer_step_layer calls over three rounds (the second with one worker
    x1000, so the decisions differ between units).  Timed units report
    positive kernel times."""
    wl = synth.small("llama1b-k8-bf16", sizes, num_workers=K, replica_dtype=dtype, name=f"pairs{name}{K}{dtype}")
    W = wl.warmup_rounds
    print(f"schedule {name}: K={K} {dtype} sizes={sizes} timing every {every}", flush=True)
    results = []
    for mode in ("layer", "round"):
        h = EditOuter(OuterConfig(K, wl.layer_numel, dtype, ema_warmup_rounds=W), DEV)
        _settle(h, wl, W)
        h.set_profiling(every)
        units = [_fresh_inputs(wl, u, 0, DEV) for u in range(wl.num_units)]
        for t in range(W, W + 3):
            std = wl.worker_std(t)
            if t == W + 1:
                std[K - 1] *= 1000.0
            for u in range(wl.num_units):
                wl.fill_replicas(units[u][0], units[u][2], u, t, std=std)
            torch.cuda.synchronize()
            if mode == "layer":
                for u in range(wl.num_units):
                    h.step_layer(u, *units[u])
            else:
                h.step_round(units)
            torch.cuda.synchronize()
            if t == W + 1:
                flagged = [h.state_get(u) for u in range(wl.num_units)]
        results.append((units, flagged + [h.state_get(u) for u in range(wl.num_units)]))
        if mode == "round" and every:
            for u in range(0, wl.num_units, every):
                p1, p2 = h.kernel_times(u)
                assert p1 > 0 and p2 > 0, f"unit {u}: kernel times {p1}, {p2}"
        h.close()
    (ua, sa), (ub, sb) = results
    for u, (a, b) in enumerate(zip(ua, ub)):
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]), f"unit {u}"
        assert all(torch.equal(x, y) for x, y in zip(a[2], b[2])), f"unit {u}"
    for x, y in zip(sa, sb):
        for f in ("norm", "ema_mean", "ema_std", "weight", "anomalous"):
            assert np.array_equal(getattr(x, f), getattr(y, f)), f
        assert x.synced_norm == y.synced_norm and x.clip_coef == y.clip_coef
    n = wl.num_units
    assert all(s.round == W + 2 for s in sb[:n]) and all(s.round == W + 3 for s in sb[n:])
    assert all(s.anomalous[K - 1] for s in sb[:n]), "the x1000 worker was not flagged in every unit"
    # on units large enough for a steady norm, the clean workers pass the z-test
    assert all(not s.anomalous[:K - 1].any() for s, size in zip(sb[:n], sizes) if size >= 10_000), \
        "a clean worker was flagged"


def test_state_get_waits_for_its_round_through_the_event_ring():
    """A round's units share one completion event from a small ring.  Seven
    rounds are enqueued on two streams without any host synchronisation
    (the ring wraps), then state_get is called at once: every unit must
    report its last round, bit for bit as a handle that synchronised after
    every round, and theta must match once the device is idle."""
    sizes = [2_000_003, 1_500_000, 2_000_000, 1_000_001, 3_000_000, 750_007]
    wl = synth.small("llama1b-k8-bf16", sizes, name="ring")
    schedule = [(0, [0, 1])] + [(1, [2, 3]), (1, [4, 5])] * 3  # (stream, units)
    results = []
    for synced in (True, False):
        h = EditOuter(OuterConfig(wl.num_workers, wl.layer_numel, "bf16"), DEV)
        units = [_fresh_inputs(wl, u, 0, DEV) for u in range(wl.num_units)]
        torch.cuda.synchronize()
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        for si, us in schedule:
            # later rounds of a unit see replicas equal to theta: zero pseudo gradients
            streams[si].wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(streams[si]):
                h.step_round([units[u] for u in us], layers=us)
            if synced:
                torch.cuda.synchronize()
        states = [h.state_get(u) for u in range(wl.num_units)]  # no synchronisation before
        torch.cuda.synchronize()
        results.append(([tuple(t.clone() for t in (x[0], x[1])) for x in units], states))
        h.close()
    (ua, sa), (ub, sb) = results
    expect_rounds = [1, 1, 3, 3, 3, 3]
    for u in range(wl.num_units):
        assert sa[u].round == sb[u].round == expect_rounds[u]
        assert np.array_equal(sa[u].norm, sb[u].norm) and np.array_equal(sa[u].ema_mean, sb[u].ema_mean)
        assert np.array_equal(sa[u].weight, sb[u].weight) and sa[u].clip_coef == sb[u].clip_coef
        assert torch.equal(ua[u][0], ub[u][0]) and torch.equal(ua[u][1], ub[u][1])


def test_round_rejects_repeated_unit():
    wl = synth.small("llama1b-k8-bf16", [4096, 4096], name="rep")
    h = EditOuter(OuterConfig(wl.num_workers, wl.layer_numel, "bf16"), DEV)
    units = [_fresh_inputs(wl, u, 0, DEV) for u in range(2)]
    with pytest.raises(EditOuterError) as e:
        h.step_round([units[0], units[0]], layers=[0, 0])
    assert "twice" in str(e.value)
    h.close()


# ------------------------------------------------------------ API errors


def test_step_rejects_bad_arguments():
    wl = synth.small("llama1b-k8-bf16", [4096, 100], name="api")
    h = EditOuter(OuterConfig(wl.num_workers, wl.layer_numel, "bf16"), DEV)
    th, b, reps = _fresh_inputs(wl, 0, 0, DEV)
    with pytest.raises(IndexError):
        h.step_layer(2, th, b, reps)
    with pytest.raises(ValueError):
        h.step_layer(0, th, b, reps[:-1])
    with pytest.raises(ValueError):
        h.step_layer(0, th, b.double(), reps)
    # misaligned pointer (offset by one element) is refused by the library
    big = torch.zeros(4097, dtype=torch.float32, device=DEV)
    with pytest.raises(EditOuterError) as e:
        h.step_layer(0, big[1:], b, reps)
    assert "aligned" in str(e.value)
    # aliasing replicas are refused
    with pytest.raises(EditOuterError) as e:
        h.step_layer(0, th, b, [reps[0]] * wl.num_workers)
    assert "overlap" in str(e.value)
    with pytest.raises(EditOuterError):
        h.state_get(1)  # never stepped
    h.close()
