"""Calls whose units have at most 64 stacked rows split each key tile between two
groups of waves: both sides of that rule, every number of 32-row blocks up to
four, prefixes whose last tile leaves the second group (keys 32-63 of a tile)
without a visible key, and a scale for which the untouched running max times the
scale would overflow."""
import numpy as np
import pytest
import torch

import gpu_util as U
import oracle
import paper_2603_01639_amd as ltd
import workloads as W

pytestmark = pytest.mark.gpu


def _check(d, G, N, prefix, block=0, scale=None):
    rng = np.random.default_rng(N * 131 + G + sum(prefix))
    trees = [W.tree_uniform_parent(rng, max(1, N - b)) for b in range(len(prefix))]
    b = W.make_batch(rng, dtype=W.DTYPE_BF16, Hq=2 * G, Hkv=2, d=d, prefix=prefix, trees=trees,
                     tokens=[W.distinct_sibling_tokens(rng, t, 600) for t in trees], Voc=600, p_match=0.7,
                     Nmax=N, block_size=block, label=f"G={G} N={N} P={prefix} block={block} scale={scale}")
    U.log(f"[key groups] d={d} {b.label}")
    dev = U.upload(b)
    out = torch.zeros(tuple(b.q.shape), dtype=torch.bfloat16, device="cuda")
    ltd.tree_verify_attn(dev.q, dev.k, dev.v, dev.prefix_len, dev.parents, dev.n_nodes, out,
                         max_prefix=b.max_prefix, block_table=dev.block_table, num_blocks=b.num_blocks,
                         scale=scale)
    want = oracle.tree_verify_attn(b.q, b.k_cache, b.v_cache, b.prefix_len, b.parents, b.n_nodes, Hkv=2,
                                   block_table=b.block_table, num_blocks=b.num_blocks, scale=scale,
                                   dtype=b.dtype)
    U.compare_attention(b, U.to_host(out), want)


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("G,N", [(1, 1), (1, 33), (4, 8), (4, 9), (8, 8), (4, 16), (1, 64), (1, 65), (5, 12),
                                 (5, 13), (4, 17), (8, 12), (4, 32), (5, 25), (5, 26), (1, 128), (1, 129)])
def test_row_counts(G, N, d):
    _check(d, G, N, [97])
    _check(d, G, N, [300, 64, 1], block=16)


@pytest.mark.parametrize("P", [0, 1, 31, 32, 33, 63, 64, 65, 96, 128, 1000])
def test_partial_tiles(P):
    _check(128, 4, 5, [P])
    _check(128, 4, 5, [P, 200], block=4)


@pytest.mark.parametrize("P", [0, 1, 31, 65])
def test_large_scale(P):
    _check(128, 4, 3, [P], scale=2.0)


@pytest.mark.parametrize("P", [256, 1024])
def test_time_of_four_row_blocks(P):
    """Two groups of waves on 128 rows made a tree of 32 nodes slower than one
    of 33, which needs a fifth block of rows."""
    rng = np.random.default_rng(P)
    calls = []
    for n in (32, 33):
        tree = W.tree_uniform_parent(rng, n)
        b = W.make_batch(rng, dtype=W.DTYPE_BF16, Hq=32, Hkv=8, d=128, prefix=[P], trees=[tree],
                         tokens=[W.distinct_sibling_tokens(rng, tree, 500)], Voc=500, p_match=0.7)
        calls.append(U.attention_call(b, P)[0])
    t = U.call_times(*calls)
    U.log(f"[key groups] P={P}: 32 nodes {t[0]:.1f} us, 33 nodes {t[1]:.1f} us")
    assert t[0] < t[1], t  # 1.16 and 1.03 times with two groups, 0.88 with one
