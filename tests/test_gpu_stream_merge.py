"""The stream plan's merge at the edges of its rows: units cut between
workgroups whose stacked rows are one less, as many and one more than a step,
a wave and a workgroup of the merge take, and a full unit."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library asks for the device)

import gpu_util as U
import workloads as W

pytestmark = pytest.mark.gpu


def _check(Hq, Hkv, d, prefix, nodes, Nmax):
    rng = np.random.default_rng(sum(nodes) + Hq + d)
    trees = [W.tree_uniform_parent(rng, n) for n in nodes]
    b = W.make_batch(rng, dtype=W.DTYPE_BF16, Hq=Hq, Hkv=Hkv, d=d, prefix=prefix, trees=trees,
                     tokens=[W.distinct_sibling_tokens(rng, t, 500) for t in trees], Voc=500, p_match=0.7,
                     Nmax=Nmax, label=f"{Hq}/{Hkv} heads, d={d}, N={nodes}")
    U.log(f"[stream merge] {b.label}")
    U.compare_attention(b, U.gpu_attention(b, U.upload(b)), U.oracle_attention(b))


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 33, 63, 64, 65, 127, 129, 255, 256])
def test_rows(n, d):
    _check(1, 1, d, [1500, 700], [n, max(1, n - 1)], 256)
