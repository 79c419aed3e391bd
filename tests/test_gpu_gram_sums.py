"""The Gram pass's sums against 64-bit torch products (GPU).

edit_outer_gram_layer returns the K(K+1)/2 sums sum_i Delta_j[i] Delta_k[i]
of a unit.  Every K has its own shape of the wave's closing reduction (an odd
number of sums pairs the last one with itself), and the unit sizes sit at the
edges of that reduction and of the loads: one element, a single lane, less
than a wave, a whole block, one more, a ragged tail, more rows than one, and
more vectors than one trip of the grid.  Each replica differs from theta by
a number of its own, so a sum that landed in another lane's place shows.

Tolerance: the products of exact fp64 differences summed in any order are
within n * 2^-52 of sum |Delta_j Delta_k| relative to it (Higham, "Accuracy
and Stability of Numerical Algorithms", Sec. 4.2: gamma_n with n additions
per order); the reference's own sums carry the same bound, so twice that.
"""
import pytest
import torch

from paper_2412_07210_amd import EditOuter, OuterConfig

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def _sizes(ve):
    return [1, ve, 63 * ve, 256 * ve, 256 * ve + 1, 300_001, 256 * 257 * ve + 5]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("K", [1, 2, 3, 4, 5, 6, 7, 8, 9, 13, 16, 17, 32])
def test_gram_sums_match_fp64_products(K, dtype):
    ve = 8 if dtype == "bf16" else 4
    sizes = _sizes(ve)
    cfg = OuterConfig(K, sizes, dtype)
    with EditOuter(cfg, DEV) as h:
        gen = torch.Generator(device=DEV).manual_seed(100 * K + ve)
        for u, n in enumerate(sizes):
            theta = torch.empty(n, device=DEV).normal_(0.0, 0.02, generator=gen)
            reps = [(theta + (j + 1) * 1e-3 * torch.empty(n, device=DEV).normal_(0.0, 1.0, generator=gen))
                    .to(cfg.torch_dtype) for j in range(K)]
            got = h.gram_layer(u, theta, reps)
            d = torch.stack([r.double() - theta.double() for r in reps])
            want, size = [], []
            for j in range(K):
                p = d[j] * d[j:]
                want.append(p.sum(1))
                size.append(p.abs().sum(1))
            want, size = torch.cat(want), torch.cat(size)
            bound = 2 * (n + 1) * 2.0 ** -52 * size
            assert bool(((got - want).abs() <= bound).all()), f"K={K} {dtype} n={n}"
