"""The split plan's merge kernels on both sides of the rule that picks between
them (at most 8 splits: 16 lanes a row; more: a wave a row) and of the splits
the wave kernel requests up front (32) and weights per lane (64)."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library asks for the device)

import gpu_util as U
import paper_2603_01639_amd as ltd
import workloads as W

pytestmark = pytest.mark.gpu


def _prefix_with_splits(splits, N, Hq, Hkv, d):
    """The shortest prefix that one sequence's plan cuts into `splits` pieces or
    more (the plan skips some counts)."""
    def grid(P):
        return ltd.attn_grid(1, N, Hq, Hkv, d, P, ltd.DTYPE_BF16, P + N)
    units = grid(1)
    for P in range(65, 12000, 16):
        if grid(P) >= units * splits:
            return P
    pytest.fail(f"no prefix gives {splits} splits")


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("splits", [3, 8, 9, 32, 33, 64, 65])
def test_split_counts(splits, d):
    Hq, Hkv, N = 8, 2, 31  # 124 rows: one row tile
    P = _prefix_with_splits(splits, N, Hq, Hkv, d)
    rng = np.random.default_rng(splits * 2 + d)
    tree = W.tree_uniform_parent(rng, N)
    b = W.make_batch(rng, dtype=W.DTYPE_BF16, Hq=Hq, Hkv=Hkv, d=d, prefix=[P], trees=[tree],
                     tokens=[W.distinct_sibling_tokens(rng, tree, 500)], Voc=500, p_match=0.7, Nmax=N + 1,
                     label=f"{splits} splits")
    U.log(f"[merge] splits={splits} d={d} P={P}")
    got = U.gpu_attention(b, U.upload(b))
    U.compare_attention(b, got, U.oracle_attention(b))
