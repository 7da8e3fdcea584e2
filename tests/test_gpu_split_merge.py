"""The split plan's merge kernels on both sides of the rule that picks between
them (at most 8 splits: 16 lanes a row; more: a wave a row), of the splits
the wave kernel requests up front (32) and of the splits it weights per lane
(64), for units of 128 rows (with two key groups and with one) and of 256."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library asks for the device)

import gpu_util as U
import paper_2603_01639_amd as ltd
import workloads as W

pytestmark = pytest.mark.gpu


def _prefix_with_splits(splits, N, Hq, Hkv, d):
    """The shortest prefix that one sequence's plan cuts into exactly `splits`
    pieces."""
    def grid(P):
        return ltd.attn_grid(1, N, Hq, Hkv, d, P, ltd.DTYPE_BF16, P + N)
    units = grid(1)
    for P in range(65, 14000, 16):
        if grid(P) == units * splits:
            return P
    pytest.fail(f"no prefix gives {splits} splits")


def _check(Hq, Hkv, N, d, P, label):
    rng = np.random.default_rng(N * 7 + P + d)
    tree = W.tree_uniform_parent(rng, N)
    b = W.make_batch(rng, dtype=W.DTYPE_BF16, Hq=Hq, Hkv=Hkv, d=d, prefix=[P], trees=[tree],
                     tokens=[W.distinct_sibling_tokens(rng, tree, 500)], Voc=500, p_match=0.7, Nmax=N, label=label)
    U.log(f"[merge] {label} d={d} P={P}")
    got = U.gpu_attention(b, U.upload(b))
    U.compare_attention(b, got, U.oracle_attention(b))


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("N,splits", [(33, 3)] + [(N, s) for N in (16, 32, 33) for s in (8, 9, 32, 33, 63, 64, 65)])
def test_split_counts(N, splits, d):
    Hq, Hkv = 8, 2  # 4 rows a node
    P = _prefix_with_splits(splits, N, Hq, Hkv, d)
    _check(Hq, Hkv, N, d, P, f"{splits} splits, {4 * N} rows")


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("P", [700, 3000])
@pytest.mark.parametrize("N", [1, 3, 4, 5, 15, 16, 17, 64, 65, 129, 255])
def test_rows(N, P, d):
    """Rows next to a multiple of 4 and of 16, a merge workgroup's: both merges
    (4 to 7 and more than 8 splits) stop after the call's rows."""
    _check(2, 2, N, d, P, f"{N} rows")
