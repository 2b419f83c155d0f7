"""GPU parity of the EM statistics for values at the ends of float32: rows of Q = G / S~ whose size changes by many orders
within a batch, between the samples that are contracted together, and Gaussian data of which some columns are tiny.  For the
former a binary tree of depth 2 whose einsum items pass entry k of both children on (one weight per output), so that the size
of every quantity is set by the leaves."""
import numpy as np
import pytest
import torch

from oracle.einet import BERNOULLI, GAUSSIAN
from tests.common import make_oracle
import workloads
from tests.gpu_common import gpu_model, dev, assert_logp_close, assert_stats_close, stat_tensors, STAT_RTOL

pytestmark = pytest.mark.gpu

VARS = 12          # per leaf


def chain_model(K):
    """Tree of depth 2, one replica; the root mixes the pairs (0, 0) and (1, 1).  Leaf probabilities of its two halves, entries
    0 and 1: 0.5 except where a set variable tells the entries apart (see batch)."""
    spec = dict(kind="rat", D=4 * VARS, depth=2, R=1)
    oracle, flat, _ = make_oracle(spec, K, 1, BERNOULLI, 5)
    g, lay = oracle.g, oracle.layout
    flat = flat.copy()
    root = next(n for n, (s, _, _) in enumerate(g.partitions) if len(g.scopes[s]) == 4 * VARS)
    for n, (s, _, _) in enumerate(g.partitions):
        w = np.zeros((1 if n == root else K, K, K), np.float32)
        if n == root:
            w[0, 0, 0] = w[0, 1, 1] = 0.5
        else:
            for k in range(K):
                w[k, k, k] = 1.0
        flat[lay.w_off[n]:lay.w_off[n] + w.size] = w.reshape(-1)
    left, right = (sorted(g.scopes[s]) for s in g.partitions[root][1:])
    phi = flat[lay.phi_off:lay.n_params].reshape(4 * VARS, K)
    phi[:] = 0.5
    phi[left[:2], 1] = 2.0 ** -15           # both set: entry 1 of the left half is 2^-28 of entry 0
    phi[right[:8], 1] = 2.0 ** -15          # all set: entry 1 of the right half is 2^-112 of entry 0
    phi[right[16:], 1] = 2.0 ** -15         # .. and these: 2^-224, zero in float32
    phi[right[8:13], 0] = 2.0 ** -13        # all set: entry 0 of it is 2^-60 of entry 1
    oracle.set_flat_params(flat)
    return spec, oracle, flat, left, right, root


def batch(kinds, left, right):
    x = np.zeros((len(kinds), 4 * VARS, 1), np.float32)
    for b, kind in enumerate(kinds):
        if kind == "large":
            x[b, left[:2]] = 1.0
            x[b, right[8:13]] = 1.0
        else:
            x[b, right[:8]] = 1.0
        if kind == "zero":
            x[b, right[16:]] = 1.0
    return x


@pytest.mark.parametrize("K,kinds", [
    (20, ["small"] * 32 + ["large"] * 128),         # shares of the batch, steps of 32 samples
    (40, ["small"] * 130 + ["large"] * 20),
    (64, ["small"] * 32 + ["large"] * 8),           # steps for any batch
    (64, ["large"] * 32 + ["small"] * 8),
    (20, ["small"] * 2 + ["large"] * 98),           # with the posteriors
    (16, ["small"] * 64 + ["large"] * 8),
])
def test_posteriors_that_grow_within_a_batch(K, kinds):
    """Entry 1 of the left half: Q is 2^-112 in "small" samples (entry 0 explains them) and 2^28 in "large" ones (entry 1
    does, and S~ is small).  Each fits float32, the quotient does not."""
    spec, oracle, flat, left, right, _ = chain_model(K)
    x = batch(kinds, left, right)
    print("growing posteriors", K, len(kinds), flush=True)
    m = gpu_model(spec, K, 1, BERNOULLI, len(kinds), 5, flat)
    ref_stats, ref_logp = oracle.em_accumulate(x)
    lp = torch.empty(len(kinds), device="cuda")
    m.em_accumulate(dev(x), None, lp)
    assert_logp_close(lp, ref_logp)
    assert_stats_close(m.stats, oracle.stats_to_flat(ref_stats), oracle.layout, m.n_params)
    m.close()


@pytest.mark.parametrize("K,kinds", [(20, ["zero"] * 64 + ["small"] * 96), (64, ["zero"] * 32 + ["small"] * 8), (64, ["small"] * 40)])
def test_smallest_posteriors_keep_their_bits(K, kinds):
    """All of an entry's posteriors are near 2^-112, or zero in the first samples: its statistics are as accurate as others
    (a quotient of two of them is a parameter).  Error of a term: four exponentials of residuals to 90, 90 * 2^-24 each."""
    spec, oracle, flat, left, right, root = chain_model(K)
    x = batch(kinds, left, right)
    print("smallest posteriors", K, len(kinds), flush=True)
    m = gpu_model(spec, K, 1, BERNOULLI, len(kinds), 5, flat)
    ref = oracle.stats_to_flat(oracle.em_accumulate(x)[0])
    m.em_accumulate(dev(x), None, None)
    got, want = (stat_tensors(f, oracle.layout, m.n_params) for f in (m.stats.cpu().numpy().astype(np.float64), ref))
    for name in ("Nw", "num", "den", "tot"):
        seen = want[name] > 2.0 ** -120
        assert np.sum(seen & (want[name] < 2.0 ** -100)) > 0
        assert np.all(np.abs(got[name] - want[name])[seen] <= STAT_RTOL * want[name][seen]), name
    m.close()


@pytest.mark.parametrize("D,depth,R,K,C,B,mask_kind", [
    (64, 1, 1, 20, 1, 300, None),                      # a tile of 16 pairs per workgroup
    (64, 1, 1, 10, 1, 300, "per_sample"),
    (1024, 1, 9, 17, 1, 140, None),                    # eight tiles per workgroup
    (1024, 1, 9, 10, 1, 140, "shared"),
])
def test_statistics_of_tiny_values(D, depth, R, K, C, B, mask_kind):
    """Columns whose values are near 1e-14 and 1e-18 throughout, beside ordinary ones, and a column with tiny values in half of
    its samples: every sum of squares is as accurate as that of ordinary values (float32: 2^-24 for each of the products and of
    the posterior's exponentials; sums over the batch of one sign)."""
    spec = dict(kind="rat", D=D, depth=depth, R=R)
    oracle, flat, rng = make_oracle(spec, K, C, GAUSSIAN, 77, leaf_range=(0.2, 0.8))
    x = workloads.draw_data(rng, dict(kind="gaussian_mixture", components=3, std=0.3), B, D, C)
    x[:, 0::5] *= np.float32(1e-14)
    x[:, 1::5] *= np.float32(1e-18)
    x[B // 2:, 2::5] *= np.float32(1e-15)
    mask = workloads.draw_mask(rng, None if mask_kind is None else dict(kind=mask_kind, observed_fraction=0.6), B, D)
    print("tiny values", D, K, B, mask_kind, flush=True)
    m = gpu_model(spec, K, C, GAUSSIAN, B, 77, flat)
    ref = oracle.stats_to_flat(oracle.em_accumulate(x, mask)[0])
    m.em_accumulate(dev(x), dev(mask), None)
    got, want = (stat_tensors(f, oracle.layout, m.n_params)["num"] for f in (m.stats.cpu().numpy().astype(np.float64), ref))
    seen = want > 2.0 ** -120
    assert want[seen].min() < 1e-30
    assert np.all(np.abs(got - want)[seen] <= STAT_RTOL * want[seen])
    m.close()
