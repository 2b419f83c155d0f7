"""Index arithmetic that kernels share with the host, run on the CPU for every launch shape: a read whose value is dropped
shows in no result, and must stay inside the caller's buffers all the same."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2004_06231_amd", "csrc")

PROGRAM = r"""
#include "kernels.hpp"
#include <cstdio>
using namespace einet_impl;

// every stage of every workgroup of an item, as k_einsum_posterior walks them
template <int K8, bool EXACT>
int walk(int K) {
    const int slices = (K + 3) / 4, sg = post_slices(K8);
    int bad = 0;
    for (int count = 1; count <= 300; ++count)
        for (int nchunks = 1; nchunks <= 8; ++nchunks) {
            const int ngr = bwd_groups_per_item(count, K, 128 * nchunks);
            for (int grp = 0; grp < ngr; ++grp)
                for (int it = grp * slices / ngr; it < (grp + 1) * slices / ngr; it += sg) {
                    for (int r = 0; r < 4 * sg; ++r) {
                        const int row = post_weight_row<K8, EXACT>(it, r, K);
                        bad += row < 0 || row >= K || (4 * it + r < K && row != 4 * it + r);
                    }
                    for (int sl = 0; sl < sg; ++sl) {
                        const int e = post_left_entry<K8, EXACT>(it + sl, K);
                        bad += (K & 3) == 0 && (e < 0 || e + 3 >= K || (4 * (it + sl) < K && e != 4 * (it + sl)));
                    }
                }
        }
    if (bad) printf("K = %d: %d reads outside the item\n", K, bad);
    return bad;
}
template <int K8>
int walk_k8() {
    int bad = walk<K8, true>(8 * K8);
    for (int K = 8 * K8 - 7; K < 8 * K8; ++K) bad += walk<K8, false>(K);
    return bad;
}
// The readers of posterior blocks find as many as the layer's workgroups write, and never more than the plan reserves.
int blocks() {
    int bad = 0;
    for (int K = 1; K <= 64; ++K)
        for (int count = 1; count <= 600; ++count)
            for (int B : {1, 2, 63, 64, 65, 127, 128, 129, 256, 257, 384, 385, 640, 1000, 4000}) {
                const int groups = bwd_groups_per_item(count, K, B), listed = bwd_groups_per_item(count, K, 1);
                int used = 0;
                for (int q = 0; q < listed; ++q) used += bwd_block_code(count, q) <= bwd_block_limit(K, B);
                bad += groups < 1 || groups > listed || used != groups ||
                       bwd_source_blocks(count, K, B) != groups;
            }
    if (bad) printf("posterior blocks: %d cases wrong\n", bad);
    return bad;
}
// Shares of the batch: whole chunks, none empty, together the batch; their blocks fit the scratch of any larger batch.
int shares() {
    int bad = 0;
    for (int K = 1; K <= 64; ++K)
        for (int count : {1, 2, 3, 4, 7, 8, 14, 16, 24, 28, 32, 48, 60, 64, 96, 97, 112, 128, 194, 384, 385, 1000, 2540})
            for (int most : {1, 128, 129, 300, 512, 1000, 4096}) {
                const size_t room = ein_stat_partial_bound(count, K, most);
                for (int B = 1; B <= most; B += most > 512 ? 37 : 1) {
                    const int n = einsum_backward_fused(count, K, B) ? fused_shares(count, K, B) : ein_stat_shares(count, K, B);
                    const int share = ein_stat_share(n, B);
                    bad += n < 1 || (long)n * share < B || (n > 1 && (share % 128 != 0 || (long)(n - 1) * share >= B ||
                                                                      (size_t)n * count * K * K * K > room));
                }
            }
    if (bad) printf("shares: %d cases wrong\n", bad);
    return bad;
}
int main() {
    if (blocks() || shares()) return 1;
    return walk_k8<3>() + walk_k8<4>() + walk_k8<5>() + walk_k8<6>() + walk_k8<7>() + walk_k8<8>() ? 1 : 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"),
                    reason="needs g++ and the HIP headers")
def test_reads_blocks_and_shares_of_the_top_down_kernels(tmp_path):
    src, exe = tmp_path / "walk.cpp", str(tmp_path / "walk")
    src.write_text(PROGRAM)
    res = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + CSRC, str(src),
                          "-o", exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-3000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout
