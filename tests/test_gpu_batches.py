"""Launches that step several units, and where their Gram input is cached (GPU).

A round steps consecutive units in batches of three launches and units of one
Gram block (at most 256 vectors) in launches of their own; the partial rows
of a unit do not depend on the batch, so every schedule must give the bits of
unit-by-unit edit_outer_step_layer calls.  The Gram pass reads the end of its
input through the cache and the rest non-temporally, two loops of the same
sums, so a step over a unit that crosses that line must give the bits of the
Gram and apply calls, which stream all of it.  Units of a round that share a
buffer are no longer independent; a round then has to give the bits of the
calls in its order.
"""
import numpy as np
import pytest
import torch

from paper_2412_07210_amd import ONE_PASS, EditOuter, OuterConfig

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def _inputs(cfg, gen):
    units = []
    for n in cfg.layer_numel:
        theta = torch.empty(n, device=DEV).normal_(0.0, 0.02, generator=gen)
        mom = torch.empty(n, device=DEV).normal_(0.0, 1e-3, generator=gen)
        reps = [(theta + (j + 1) * 1e-3 * torch.empty(n, device=DEV).normal_(0.0, 1.0, generator=gen))
                .to(cfg.torch_dtype) for j in range(cfg.num_workers)]
        units.append((theta, mom, reps))
    return units


def _copy(units):
    return [(t.clone(), b.clone(), [r.clone() for r in reps]) for t, b, reps in units]


def _same(a, b, what):
    for u, (x, y) in enumerate(zip(a, b)):
        assert torch.equal(x[0], y[0]) and torch.equal(x[1], y[1]), f"{what}: unit {u}"
        assert all(torch.equal(p, q) for p, q in zip(x[2], y[2])), f"{what}: unit {u} replicas"


def _same_state(a, b, n, what):
    for u in range(n):
        x, y = a.state_get(u), b.state_get(u)
        for f in ("norm", "ema_mean", "ema_std", "weight", "anomalous"):
            assert np.array_equal(getattr(x, f), getattr(y, f)), f"{what}: unit {u} {f}"
        assert (x.synced_norm, x.clip_coef, x.round) == (y.synced_norm, y.clip_coef, y.round), f"{what}: unit {u}"


# vectors per unit: single blocks (0..256), the first of two rows (257), one
# row per CU and one vector more (65,536, 65,537), and 18 units of more than
# one block, which no batch holds; "ragged" elements follow the last vector
_MIXES = {
    "all small": [0, 1, 255, 256, 3, 17, 256, 2, 9, 100, 31, 64, 65, 5, 7, 8, 250, 11, 256],
    "full batch": [257 + 16 * i for i in range(16)],
    "past a batch": [300, 257, 65_537, 400, 999, 1000, 258, 513, 65_536, 270, 301, 800, 4097, 600, 512, 2049, 700,
                     9_999],
    "mixed": [1000, 3, 70_000, 0, 257, 256, 1, 5000],
}


@pytest.mark.parametrize("K,dtype", [(1, "f32"), (4, "f32"), (8, "bf16"), (9, "bf16"), (16, "f32"), (17, "bf16"),
                                     (32, "bf16")])
@pytest.mark.parametrize("mix", list(_MIXES))
def test_round_in_batches_matches_unit_by_unit(mix, K, dtype):
    ve = 8 if dtype == "bf16" else 4
    sizes = [v * ve + i % ve for i, v in enumerate(_MIXES[mix])]
    cfg = OuterConfig(K, sizes, dtype, clip_threshold=0.05)
    gen = torch.Generator(device=DEV).manual_seed(K)
    one = _inputs(cfg, gen)
    all_ = _copy(one)
    with EditOuter(cfg, DEV) as a, EditOuter(cfg, DEV) as b:
        for _ in range(2):  # the second round starts from equal replicas
            for u, unit in enumerate(one):
                a.step_layer(u, *unit)
            b.step_round(all_)
        torch.cuda.synchronize()
        _same(one, all_, f"{mix} K={K} {dtype}")
        _same_state(a, b, len(sizes), f"{mix} K={K} {dtype}")


@pytest.mark.parametrize("K,dtype,sizes", [
    # a batch's last 160 MB of Gram input are read through the cache: the line
    # falls into the first of three units, the second of four, between two
    (8, "bf16", [12_000_005, 3_000_000, 1_000_003]),
    (4, "f32", [3_000_001, 4_000_002, 2_500_000, 3_500_003]),
    (1, "f32", [6_000_000, 10_000_000, 10_000_000]),
    # the third unit would take the batch past 4 GiB
    (2, "bf16", [200_000_001, 200_000_002, 200_000_003]),
    # units that take a batch of their own (over 240 MiB bf16, 768 MiB fp32),
    # first, between and behind others
    (12, "bf16", [9_000_001, 1_000_000, 700_001, 9_000_002, 9_000_003, 3]),
    (16, "f32", [400_000, 12_000_001, 300_001]),
])
def test_round_across_the_byte_limits_matches_unit_by_unit(K, dtype, sizes):
    cfg = OuterConfig(K, sizes, dtype, clip_threshold=0.05)
    one = _inputs(cfg, torch.Generator(device=DEV).manual_seed(K))
    all_ = _copy(one)
    with EditOuter(cfg, DEV) as a, EditOuter(cfg, DEV) as b:
        for u, unit in enumerate(one):
            a.step_layer(u, *unit)
        b.step_round(all_)
        torch.cuda.synchronize()
        _same(one, all_, f"K={K} {dtype}")
        _same_state(a, b, len(sizes), f"K={K} {dtype}")


# (unit, buffer) that is a piece of (another unit, buffer) from the given
# vector on; buffers: 0 theta, 1 momentum, 2.. replicas.  Sizes in vectors.
_TIES = {
    "large with large": ([600, 700, 600, 500], [(2, b, 0, b, 0) for b in range(3)]),
    "piece of the one before": ([5000, 4000, 3000, 300], [(1, 3, 0, 3, 1000), (2, 0, 1, 0, 7), (3, 1, 2, 1, 2700)]),
    "small with large": ([900, 100, 256, 800, 400], [(1, 0, 0, 0, 800), (2, 3, 3, 3, 100), (1, 1, 4, 1, 7)]),
    "small with small": ([200, 150, 256, 1, 40], [(1, 1, 0, 1, 50), (1, 2, 2, 2, 90), (4, 0, 2, 0, 216)]),
    "past a full batch": ([300 + u for u in range(18)] + [20 + u for u in range(20)],
                          [(16, 1, 17, 1, 1), (1, 2, 16, 2, 3), (19, 0, 37, 0, 5), (36, 3, 2, 3, 10)]),
}


@pytest.mark.parametrize("every", [0, 3])
@pytest.mark.parametrize("K,dtype", [(4, "f32"), (8, "bf16"), (16, "bf16"), (17, "f32")])
@pytest.mark.parametrize("ties", list(_TIES))
def test_round_with_shared_buffers_matches_unit_by_unit(ties, K, dtype, every):
    """Also with kernel timing on every third unit, whose launches go ahead of
    the units that wait."""
    ve = 8 if dtype == "bf16" else 4
    vecs, shared = _TIES[ties]
    sizes = [v * ve for v in vecs]
    cfg = OuterConfig(K, sizes, dtype, clip_threshold=0.05)

    def units():
        made = [[t, b, *reps] for t, b, reps in _inputs(cfg, torch.Generator(device=DEV).manual_seed(K))]
        for u, buf, of, of_buf, at in shared:
            made[u][buf] = made[of][of_buf][at * ve:at * ve + sizes[u]]
            assert made[u][buf].numel() == sizes[u]
        return [(m[0], m[1], m[2:]) for m in made]

    one, all_ = units(), units()
    with EditOuter(cfg, DEV) as a, EditOuter(cfg, DEV) as b:
        b.set_profiling(every)
        for _ in range(2):
            for u, unit in enumerate(one):
                a.step_layer(u, *unit)
            b.step_round(all_)
        torch.cuda.synchronize()
        _same(one, all_, f"{ties} K={K} {dtype}")
        _same_state(a, b, len(sizes), f"{ties} K={K} {dtype}")


@pytest.mark.parametrize("K,dtype,n", [(8, "bf16", 12_000_005), (4, "f32", 9_000_003), (2, "bf16", 25_000_001),
                                       (1, "f32", 25_000_002)])
def test_step_across_the_cached_end_matches_the_streamed_gram(K, dtype, n):
    cfg = OuterConfig(K, [n], dtype)
    gen = torch.Generator(device=DEV).manual_seed(n)
    one = _inputs(cfg, gen)
    two = _copy(one)
    with EditOuter(cfg, DEV) as a, EditOuter(cfg, DEV) as b:
        a.step_layer(0, *one[0])
        theta, mom, reps = two[0]
        b.apply_layer(0, b.gram_layer(0, theta, reps), theta, mom, reps)
        torch.cuda.synchronize()
        _same(one, two, f"K={K} {dtype} n={n}")
        _same_state(a, b, 1, f"K={K} {dtype} n={n}")


@pytest.mark.parametrize("K,dtype,rows", [(16, "f32", 7710), (16, "f32", 7711), (32, "bf16", 3972), (24, "bf16", 9999)])
def test_one_pass_norms_on_both_sides_of_the_fold(K, dtype, rows):
    """Past 131,072 doubles of partial rows a one-pass unit's rows are summed
    in slices first: G_j and ||Delta_bar|| of a step alone and of a round,
    against 64-bit torch sums (n * 2^-52 relative, all terms positive)."""
    per_row = 64 * (8 if dtype == "bf16" else 4) * (2 if dtype == "bf16" and K <= 16 else 1)
    n = (rows - 1) * per_row + 3
    cfg = OuterConfig(K, [n, 1000, n], dtype, flags=ONE_PASS)
    gen = torch.Generator(device=DEV).manual_seed(rows)
    units = _inputs(cfg, gen)
    want = []
    for t, _, reps in units:
        d = torch.stack([r.double() - t.double() for r in reps])
        want.append((d.square().sum(1).sqrt(), d.mean(0).square().sum().sqrt()))
        del d
    with EditOuter(cfg, DEV) as h:
        h.step_layer(0, *units[0])
        h.step_round(units[1:], layers=[1, 2])
        for u, (g, bar) in enumerate(want):
            st = h.state_get(u)
            m = cfg.layer_numel[u]
            assert np.allclose(st.norm, g.cpu().numpy(), rtol=(m + 1) * 2.0 ** -52, atol=0.0), f"unit {u}"
            assert abs(st.synced_norm - float(bar)) <= (m + K) * 2.0 ** -52 * float(bar), f"unit {u}"
            assert st.round == 1
