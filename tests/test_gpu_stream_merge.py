"""The stream plan's merge at the edges of its rows: units cut between
workgroups whose stacked rows are one less, as many and one more than a step,
a wave and a workgroup of the merge take, and a full unit."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library asks for the device)

import gpu_util as U
import workloads as W

pytestmark = pytest.mark.gpu


def _check(Hq, Hkv, d, prefix, nodes, Nmax, block=0):
    rng = np.random.default_rng(sum(nodes) + Hq + d)
    trees = [W.tree_uniform_parent(rng, n) for n in nodes]
    b = W.make_batch(rng, dtype=W.DTYPE_BF16, Hq=Hq, Hkv=Hkv, d=d, prefix=prefix, trees=trees,
                     tokens=[W.distinct_sibling_tokens(rng, t, 500) for t in trees], Voc=500, p_match=0.7,
                     Nmax=Nmax, block_size=block, label=f"{Hq}/{Hkv} heads, d={d}, N={nodes}")
    U.log(f"[stream merge] {b.label}")
    U.compare_attention(b, U.gpu_attention(b, U.upload(b)), U.oracle_attention(b))


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 33, 63, 64, 65, 127, 129, 255, 256])
def test_rows(n, d):
    _check(1, 1, d, [1500, 700], [n, max(1, n - 1)], 256)


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("B", [127, 128])
def test_wide_table(B, d):
    """Both sides of the 2048 units (16 a sequence here) from which a wave of
    the merge takes 16 rows."""
    _check(64, 8, d, [37 * (i % 7) for i in range(B)], [1 + (5 * i) % 33 for i in range(B)], 33)


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("n", [1, 3, 4, 13, 51, 52])
def test_rows_of_a_wide_table(n, d):
    """The row edges (5 rows a node) in a table of 2048 units of which few are
    cut: two longer sequences, the others of one key."""
    B = 128
    _check(40, 8, d, [900, 500] + [0] * (B - 2), [n, max(1, n - 1)] + [1] * (B - 2), 52, block=16)


def test_time_of_many_pieces():
    """Two rows a lane in every batch of pieces made the merge of units of about
    128 pieces as slow for 64 dims as for 128."""
    calls = []
    for d in (64, 128):
        rng = np.random.default_rng(d)
        trees = [W.tree_uniform_parent(rng, n) for n in (5, 2)]
        b = W.make_batch(rng, dtype=W.DTYPE_BF16, Hq=8, Hkv=1, d=d, prefix=[3243, 4681], trees=trees,
                         tokens=[W.distinct_sibling_tokens(rng, t, 500) for t in trees], Voc=500, p_match=0.7,
                         Nmax=256)
        calls.append(U.attention_call(b, 18724)[0])
    t = U.call_times(*calls)
    U.log(f"[stream merge] many pieces: 64 dims {t[0]:.1f} us, 128 dims {t[1]:.1f} us")
    assert t[0] < 0.87 * t[1], t  # 0.94 with two rows a lane, 0.78 with one
