"""GPU parity of the EM statistics where the kernels of the top-down pass change over: weight statistics formed with the
posteriors (K to 16, batches to 64, an item in one workgroup or its slices over several; K 17 to 48, chunks of the batch with a
block each or in turn), in a launch of their own from a whole batch at once (to 128 samples) or step by step, and over shares of
the batch; leaf statistics entry by entry (below 16 (variable, channel) pairs), with a tile of 16
pairs per workgroup (to 512 tiles) or with eight, with and without flags, from assembled posteriors and from the parents'
blocks; the bottom-up kernel for small items with several chunks of 64 samples per workgroup and with an item's outputs
dealt to several workgroups.  The tolerance is the one of the statistics everywhere: float32 rounding of sums over the batch,
which the products of split operands (error 2^-24 of each) do not exceed."""
import pytest
import torch

import workloads
from oracle.einet import BERNOULLI, GAUSSIAN
from tests.common import make_oracle
from tests.gpu_common import gpu_model, dev, assert_logp_close, assert_stats_close

pytestmark = pytest.mark.gpu


def rat(D, depth, R):
    return dict(kind="rat", D=D, depth=depth, R=R)


CASES = [
    # spec, K, C, family, B, mask kind, leaf range
    (rat(30, 1, 1), 10, 1, BERNOULLI, 64, None, (0.1, 0.9)),               # scopes of 15 pairs: entry by entry
    (rat(32, 1, 1), 10, 1, BERNOULLI, 65, None, (0.1, 0.9)),               # 16 pairs: one full tile; two steps, the second of one sample
    (rat(34, 1, 2), 17, 1, GAUSSIAN, 33, "per_sample", (0.2, 0.8)),        # 17 pairs: a tile of one; K = 17
    (rat(66, 1, 2), 32, 3, GAUSSIAN, 257, "shared", (0.2, 0.8)),           # the batch goes round the eight waves once and one
    (rat(40, 1, 1), 64, 1, GAUSSIAN, 40, "per_sample", (0.2, 0.8)),        # all columns, three kinds of sums
    (rat(1100, 5, 9), 7, 1, GAUSSIAN, 70, "per_sample", (0.2, 0.8)),       # 288 leaves of 34 and 35 pairs: 864 tiles, eight per workgroup
    (rat(1100, 5, 9), 33, 1, GAUSSIAN, 5, None, (0.2, 0.8)),               # the same without flags, columns beyond two tiles
    (dict(kind="pd", H=8, W=8, deltas=[4, 2]), 16, 4, GAUSSIAN, 64, "shared", (0.2, 0.8)),   # 16 pairs, assembled posteriors
    (dict(kind="pd", H=8, W=8, deltas=[2]), 41, 4, GAUSSIAN, 128, None, (0.2, 0.8)),         # the longest batch taken at once
    (dict(kind="pd", H=8, W=8, deltas=[2]), 36, 4, GAUSSIAN, 129, None, (0.2, 0.8)),         # one more
    (rat(32, 4, 12), 4, 1, BERNOULLI, 64, None, (0.1, 0.9)),               # statistics with the posteriors
    (rat(32, 4, 12), 3, 1, BERNOULLI, 65, None, (0.1, 0.9)),               # in a launch of their own; pieces that overlap
    (rat(64, 5, 16), 9, 1, BERNOULLI, 1100, None, (0.1, 0.9)),             # 256 items, 18 chunks: three chunks per workgroup
    (rat(16, 2, 1), 16, 1, BERNOULLI, 1, None, (0.1, 0.9)),                # an item's outputs over four workgroups
    (rat(32, 2, 2), 20, 1, GAUSSIAN, 900, None, (0.2, 0.8)),               # four items: shares of the batch, the last ragged
    (rat(16, 2, 1), 24, 1, GAUSSIAN, 128, None, (0.2, 0.8)),               # K from 17, one chunk: posteriors and statistics in one launch
    (rat(16, 2, 1), 21, 1, GAUSSIAN, 129, None, (0.2, 0.8)),               # one more, rows read entry by entry: a block per chunk
    (dict(kind="pd", H=6, W=6, deltas=[2]), 29, 1, GAUSSIAN, 50, None, (0.2, 0.8)),          # the same, from assembled posteriors
    (rat(16, 2, 1), 37, 1, GAUSSIAN, 20, None, (0.2, 0.8)),                # the same, three column tiles
    (dict(kind="pd", H=6, W=6, deltas=[2]), 20, 1, GAUSSIAN, 65, None, (0.2, 0.8)),          # whole items bottom-up, a second chunk of one sample
    (rat(16, 2, 1), 20, 1, BERNOULLI, 1, None, (0.1, 0.9)),                # its outputs over five workgroups
    (rat(64, 5, 16), 13, 1, BERNOULLI, 129, None, (0.1, 0.9)),             # split operands bottom-up: 256 items, two chunks
    (rat(600, 2, 2), 24, 1, BERNOULLI, 150, None, (1e-6, 1.0 - 1e-6)),     # posteriors and S~ over hundreds of binary orders
    (rat(64, 3, 20), 20, 1, GAUSSIAN, 200, None, (0.2, 0.8)),              # 120 items in one launch per layer, a block per chunk
    (rat(64, 2, 32), 28, 1, GAUSSIAN, 129, None, (0.2, 0.8)),              # 64 items, both chunks in turn, the second of one sample
    (rat(64, 2, 32), 22, 1, GAUSSIAN, 129, None, (0.2, 0.8)),              # as many items, a block per chunk, rows read entry by entry
    (rat(64, 3, 32), 24, 1, GAUSSIAN, 257, None, (0.2, 0.8)),              # three chunks of 192 items: statistics in a launch of their own
    (rat(16, 2, 12), 32, 1, GAUSSIAN, 385, None, (0.2, 0.8)),              # 24 items, four blocks each
    (rat(16, 2, 13), 32, 1, GAUSSIAN, 513, None, (0.2, 0.8)),              # 26 items, five blocks each
    (rat(16, 2, 12), 44, 1, GAUSSIAN, 300, None, (0.2, 0.8)),              # 24 items, K from 41, three blocks each
    (rat(16, 2, 12), 40, 1, GAUSSIAN, 400, None, (0.2, 0.8)),              # the same, a chunk more: statistics in a launch of their own
    (rat(16, 2, 2), 44, 1, GAUSSIAN, 33, None, (0.2, 0.8)),                # one launch per layer, K from 41
    (rat(16, 2, 1), 48, 1, GAUSSIAN, 150, None, (0.2, 0.8)),               # the same, a block per chunk
    (rat(16, 2, 1), 49, 1, GAUSSIAN, 40, None, (0.2, 0.8)),                # beyond it: in a launch of their own
    (rat(16, 2, 1), 56, 1, GAUSSIAN, 300, None, (0.2, 0.8)),               # the same, over shares of the batch
    (rat(16, 2, 1), 16, 1, BERNOULLI, 700, None, (0.1, 0.9)),              # K to 16, few items, many samples: shares of the batch
    (rat(32, 2, 2), 7, 1, BERNOULLI, 513, None, (0.1, 0.9)),               # the same, the last share of one sample, pieces that overlap
    (dict(kind="pd", H=6, W=6, deltas=[2]), 13, 1, GAUSSIAN, 64, None, (0.2, 0.8)),   # K 9 to 16, to 64 samples: an item's slices over several workgroups
    (rat(64, 5, 16), 15, 1, BERNOULLI, 63, None, (0.1, 0.9)),              # many items: one workgroup each
    (rat(1100, 5, 9), 7, 1, GAUSSIAN, 20, "per_sample", (0.2, 0.8)),       # eight tiles per workgroup, part of a step
]


@pytest.mark.parametrize("spec,K,C,family,B,mask_kind,leaf_range", CASES)
def test_statistics_where_kernels_change_over(spec, K, C, family, B, mask_kind, leaf_range):
    print("top-down edge case", spec, K, C, family, B, mask_kind, flush=True)
    seed = 9000 + K + B
    oracle, flat, rng = make_oracle(spec, K, C, family, seed, leaf_range=leaf_range)
    D = oracle.g.num_vars
    x = workloads.draw_data(rng, dict(kind="bernoulli_iid", p=0.4) if family == BERNOULLI
                            else dict(kind="gaussian_mixture", components=3, std=0.3), B, D, C)
    mask = workloads.draw_mask(rng, None if mask_kind is None else dict(kind=mask_kind, observed_fraction=0.6), B, D)
    m = gpu_model(spec, K, C, family, B, seed, flat)
    ref_stats, ref_logp = oracle.em_accumulate(x, mask)
    ref_flat = oracle.stats_to_flat(ref_stats)
    lp = torch.empty(B, device="cuda")
    m.em_accumulate(dev(x), dev(mask), lp)
    assert_logp_close(lp, ref_logp)
    assert_stats_close(m.stats, ref_flat, oracle.layout, m.n_params)
    m.em_accumulate(dev(x), dev(mask), lp)               # added to
    assert_stats_close(m.stats, 2.0 * ref_flat, oracle.layout, m.n_params)
    m.close()
