"""GPU parity at the sizes where a kernel's tiles, passes and dispatch rules have their edges: an E-step, the same E-step
added to it, and an M-step against the float64 oracle."""
import numpy as np
import pytest
import torch

import workloads
from oracle.einet import BERNOULLI, BINOMIAL, CATEGORICAL, GAUSSIAN
from tests.common import make_oracle
from tests.gpu_common import gpu_model, dev, assert_logp_close, assert_stats_close

pytestmark = pytest.mark.gpu


def _check(family, param, spec, K, C, B, mask_kind, seed, stat_rtol=1e-3, atol_rel=1e-6):
    oracle, flat, rng = make_oracle(spec, K, C, family, seed, (0.2, 0.8), leaf_param=param)
    D = oracle.g.num_vars
    data = {GAUSSIAN: dict(kind="gaussian_mixture", components=3, std=0.3),
            BERNOULLI: dict(kind="bernoulli_iid", p=0.4),
            BINOMIAL: dict(kind="binomial_mixture", components=3, trials=param, lo=0.1, hi=0.9),
            CATEGORICAL: dict(kind="categorical_mixture", components=3, values=param)}[family]
    x = workloads.draw_data(rng, data, B, D, C)
    mask = workloads.draw_mask(rng, None if mask_kind is None else dict(kind=mask_kind, observed_fraction=0.6), B, D)
    m = gpu_model(spec, K, C, family, B, seed, flat, param)
    ref_stats, ref_logp = oracle.em_accumulate(x, mask)
    ref_flat = oracle.stats_to_flat(ref_stats)
    assert_logp_close(m.logp(dev(x), dev(mask)), ref_logp)
    lp = torch.empty(B, device="cuda")
    m.em_accumulate(dev(x), dev(mask), lp)
    assert_logp_close(lp, ref_logp)
    assert_stats_close(m.stats, ref_flat, oracle.layout, m.n_params, stat_rtol, atol_rel)
    m.em_accumulate(dev(x), dev(mask), lp)               # added to, not overwritten
    assert_stats_close(m.stats, 2.0 * ref_flat, oracle.layout, m.n_params, stat_rtol, atol_rel)
    kw = dict(step=0.6, w_floor=1e-9)
    m.em_update(**kw)
    oracle.em_update(ref_stats, **kw)                    # (the M-step does not depend on the scale of the statistics)
    got, ref = m.params.cpu().numpy().astype(np.float64), oracle.get_flat_params()
    assert np.all(np.isfinite(got))
    assert np.all(np.abs(got - ref) <= 1e-3 * np.abs(ref) + 1e-7)
    m.close()


# tables of 16, 32, 64, 128 and 256 values, entries in tiles of 16, four pairs per workgroup, passes of 128 samples
@pytest.mark.parametrize("V,spec,K,C,B,mask_kind", [
    (16, dict(kind="rat", D=20, depth=2, R=2), 16, 1, 128, None),
    (17, dict(kind="pd", H=5, W=5, deltas=[3]), 17, 1, 129, "shared"),
    (33, dict(kind="rat", D=13, depth=2, R=3), 15, 3, 33, "per_sample"),
    (65, dict(kind="pd", H=4, W=6, deltas=[2]), 33, 1, 31, None),
    (129, dict(kind="rat", D=9, depth=1, R=1), 64, 2, 257, "per_sample"),
    (256, dict(kind="pd", H=6, W=6, deltas=[3]), 1, 1, 1, None),
    # M-step: a column per thread up to eight values, shared columns beyond; several (variable, replica) pairs per workgroup
    # with some left over, one pair with threads left over
    (2, dict(kind="rat", D=21, depth=2, R=3), 10, 3, 33, "per_sample"),
    (8, dict(kind="rat", D=11, depth=2, R=2), 64, 1, 40, None),
    (9, dict(kind="rat", D=13, depth=2, R=3), 17, 2, 20, None),
    (255, dict(kind="rat", D=7, depth=1, R=2), 3, 1, 60, "shared"),
    (100, dict(kind="pd", H=4, W=4, deltas=[2]), 40, 1, 50, None),
])
def test_categorical_statistics_edges(V, spec, K, C, B, mask_kind):
    print("categorical statistics", V, spec, K, C, B, mask_kind, flush=True)
    _check(CATEGORICAL, V, spec, K, C, B, mask_kind, 300 + V)


# Bottom-up einsum kernels: K around the widths of the operands (up to 8, 9 .. 16, 17 .. 20, 21 .. 32, up to 40, above), chunks
# of 128 samples and waves of 32, launches on both sides of the rules (items, samples), several chunks per workgroup.
# All operands are positive, so the relative error of a sum is that of its terms (2^-24 each) and of the exponentials
# (about 1e-6 for exponents up to 10): 3e-5 leaves a factor of ten.
@pytest.mark.parametrize("spec,K,C,B,mask_kind", [
    (dict(kind="rat", D=24, depth=3, R=2), 8, 1, 129, None),            # specialised waves, float32
    (dict(kind="rat", D=12, depth=2, R=140), 8, 1, 130, None),          # a workgroup per four outputs: many items
    (dict(kind="rat", D=24, depth=3, R=2), 9, 1, 127, "shared"),
    (dict(kind="rat", D=12, depth=2, R=40), 9, 1, 33, None),            # many items, few samples: the float32 kernel
    (dict(kind="rat", D=12, depth=2, R=70), 10, 1, 1100, None),         # two chunks per workgroup, the last one of 76 samples
    (dict(kind="rat", D=12, depth=2, R=80), 13, 1, 1025, "per_sample"),  # ... of a single sample, a chunk of its own
    (dict(kind="rat", D=12, depth=2, R=40), 13, 1, 300, None),
    (dict(kind="pd", H=6, W=6, deltas=[2]), 16, 1, 33, "per_sample"),
    (dict(kind="pd", H=6, W=6, deltas=[2]), 16, 1, 65, None),
    (dict(kind="pd", H=6, W=6, deltas=[2]), 17, 1, 1, None),
    (dict(kind="rat", D=12, depth=2, R=40), 18, 1, 260, None),          # many items: the float32 kernel
    (dict(kind="rat", D=12, depth=2, R=40), 18, 1, 520, None),          # ... with more than four chunks: persistent
    (dict(kind="pd", H=6, W=6, deltas=[2]), 20, 1, 140, None),
    (dict(kind="rat", D=24, depth=3, R=2), 24, 1, 129, None),           # specialised waves, float32
    (dict(kind="rat", D=24, depth=3, R=2), 24, 1, 5, None),
    (dict(kind="rat", D=12, depth=2, R=40), 24, 1, 129, None),          # persistent
    (dict(kind="pd", H=4, W=6, deltas=[2]), 25, 3, 64, None),
    (dict(kind="rat", D=12, depth=2, R=40), 28, 1, 20, None),           # the float32 kernel between two counts of items
    (dict(kind="rat", D=12, depth=2, R=40), 31, 1, 140, None),          # persistent: more than 1024 units
    (dict(kind="pd", H=4, W=6, deltas=[2]), 32, 1, 257, "shared"),
    (dict(kind="pd", H=4, W=6, deltas=[2]), 33, 1, 100, None),
    (dict(kind="pd", H=4, W=6, deltas=[2]), 36, 1, 100, None),          # the float32 kernel
    (dict(kind="rat", D=16, depth=2, R=3), 39, 1, 130, None),
    (dict(kind="rat", D=16, depth=2, R=70), 40, 1, 2, None),
    (dict(kind="pd", H=4, W=6, deltas=[2]), 41, 1, 33, None),
    (dict(kind="rat", D=16, depth=2, R=3), 48, 1, 64, None),            # a workgroup per four outputs
    (dict(kind="rat", D=16, depth=2, R=3), 48, 1, 257, "shared"),       # specialised waves, float32
])
def test_einsum_forward_edges(spec, K, C, B, mask_kind):
    print("einsum forward", spec, K, C, B, mask_kind, flush=True)
    _check(GAUSSIAN, 0, spec, K, C, B, mask_kind, 600 + K, stat_rtol=3e-5)


# Items with a single output entry in the kernels of the inner layers: a root with more partitions than its own kernel takes.
@pytest.mark.parametrize("R,K,B", [(3300, 13, 70), (3300, 16, 5), (3100, 18, 3), (2900, 22, 5), (2900, 24, 66), (2300, 36, 3),
                                   (2300, 40, 2)])
def test_many_root_partitions(R, K, B):
    print("many root partitions", R, K, B, flush=True)
    _check(GAUSSIAN, 0, dict(kind="rat", D=4, depth=1, R=R), K, 1, B, None, 800 + K, stat_rtol=3e-5)


# Leaf layer for short scopes and many outputs (at least a million): K around its register sizes 8, 16, 32, 64 and not a
# multiple of four, workgroups of 128 samples that are full, nearly empty and one short, several channels, both masks.
# The sums are float64 as in the oracle, so the log-densities are held to the suite's tolerance and nothing else.
@pytest.mark.parametrize("family,param,spec,K,C,B,mask_kind", [
    (BINOMIAL, 255, dict(kind="rat", D=40, depth=4, R=40), 10, 1, 200, None),
    (BINOMIAL, 7, dict(kind="rat", D=24, depth=3, R=150), 8, 2, 129, "per_sample"),
    (BERNOULLI, 0, dict(kind="rat", D=32, depth=5, R=520), 1, 1, 64, "shared"),
    (BERNOULLI, 0, dict(kind="rat", D=20, depth=2, R=20), 64, 1, 257, None),
    (GAUSSIAN, 0, dict(kind="rat", D=16, depth=2, R=30), 33, 3, 255, "per_sample"),
    (GAUSSIAN, 0, dict(kind="rat", D=30, depth=3, R=60), 17, 1, 128, None),
    # few entries of one or two variables: a thread per entry again beyond one chunk of samples
    (BERNOULLI, 0, dict(kind="rat", D=64, depth=5, R=160), 1, 1, 200, "per_sample"),
    (GAUSSIAN, 0, dict(kind="rat", D=32, depth=5, R=160), 3, 1, 129, None),
    (GAUSSIAN, 0, dict(kind="rat", D=32, depth=5, R=160), 4, 1, 129, None),
])
def test_short_leaf_edges(family, param, spec, K, C, B, mask_kind):
    print("short leaves", family, spec, K, C, B, mask_kind, flush=True)
    oracle, flat, rng = make_oracle(spec, K, C, family, 900 + K, (0.2, 0.8), leaf_param=param)
    D = oracle.g.num_vars
    data = {GAUSSIAN: dict(kind="gaussian_mixture", components=3, std=0.3), BERNOULLI: dict(kind="bernoulli_iid", p=0.4),
            BINOMIAL: dict(kind="binomial_mixture", components=3, trials=param, lo=0.1, hi=0.9)}[family]
    x = workloads.draw_data(rng, data, B, D, C)
    mask = workloads.draw_mask(rng, None if mask_kind is None else dict(kind=mask_kind, observed_fraction=0.6), B, D)
    m = gpu_model(spec, K, C, family, B, 900 + K, flat, param)
    assert_logp_close(m.logp(dev(x), dev(mask)), oracle.logp(x, mask))
    m.close()


# Weights down to the smallest normal float32 (an M-step without a floor reaches them): a sum that consists of such a weight
# alone must be as good as one of ordinary weights.  Only entry 1 of a leaf allows the value 1, and all pairs of entries but
# (0, 0) have weights of 2^-125 to 2^-124, so the sum of every inner entry is the weight of the pair (1, 1).  Its float32
# logarithm is near -86 (rounding 4e-6, twice per path), the log-density near -170 (rounding 8e-6).
@pytest.mark.parametrize("K,R,B", [(9, 2, 5), (10, 2, 64), (16, 2, 129), (18, 2, 33), (24, 2, 130), (30, 2, 64),
                                   (18, 110, 129), (36, 2, 64), (40, 2, 129)])
def test_smallest_weights_keep_their_bits(K, R, B):
    print("smallest weights", K, R, B, flush=True)
    spec = dict(kind="rat", D=8, depth=2, R=R)
    oracle, flat, rng = make_oracle(spec, K, 1, BERNOULLI, 700 + K, (0.2, 0.8))
    flat = flat.copy()
    g, lay = oracle.g, oracle.layout
    for n, (parent, _, _) in enumerate(g.partitions):
        if g.k_out(parent, K) == K:
            w = np.ldexp(rng.uniform(1.0, 2.0, (K, K, K)), -125)
            w[:, 0, 0] = 1.0
            flat[lay.w_off[n]:lay.w_off[n] + K ** 3] = w.ravel()
    phi = flat[lay.phi_off:lay.phi_off + g.num_vars * g.num_replica * K].reshape(g.num_vars, g.num_replica, K)
    phi[:, :, 0] = 0.0
    phi[:, :, 2:] = 0.0
    oracle.set_flat_params(flat)
    m = gpu_model(spec, K, 1, BERNOULLI, B, 700 + K, flat)
    got = m.logp(torch.ones(B, 8, 1, device="cuda")).cpu().numpy().astype(np.float64)
    ref = oracle.logp(np.ones((B, 8, 1)))
    assert np.all(np.abs(got - ref) <= 5e-5), np.abs(got - ref).max()
    m.close()
