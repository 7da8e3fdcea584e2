"""Calls whose bounds (Nmax, max_prefix) are far above their data, as a decoder
makes them whose buffers are sized once: attention results against the oracle,
with a workspace full of NaN so that a partial nobody wrote shows, and times
against the same call with tight bounds."""
import numpy as np
import pytest
import torch

import gpu_util as U
import paper_2603_01639_amd as ltd
import workloads as W

pytestmark = pytest.mark.gpu


def _batch(Hq, Hkv, d, prefix, nodes, Nmax, block=0):
    rng = np.random.default_rng(sum(prefix) * 31 + sum(nodes))
    trees = [W.tree_uniform_parent(rng, n) for n in nodes]
    return W.make_batch(rng, dtype=W.DTYPE_BF16, Hq=Hq, Hkv=Hkv, d=d, prefix=prefix, trees=trees,
                        tokens=[W.distinct_sibling_tokens(rng, t, 500) for t in trees], Voc=500, p_match=0.7,
                        Nmax=Nmax, block_size=block, label=f"d={d} P={prefix} N={nodes} Nmax={Nmax}")


def _check(b, max_prefix):
    U.log(f"[loose bounds] {b.label} max_prefix={max_prefix}")
    run, out = U.attention_call(b, max_prefix)
    run()
    U.compare_attention(b, U.to_host(out), U.oracle_attention(b))


@pytest.mark.parametrize("d", [128, 64])
def test_more_workgroups_than_items(d):
    """The stream plan sized for 256-node trees, given tiny ones: most
    workgroups own no item, and a unit's pieces lie between them (the first
    batch's long unit spans about 150 workgroups, more than one wave's lanes)."""
    _check(_batch(8, 1, d, [2000, 0, 0, 0], [1, 1, 1, 1], 256), 2048)
    _check(_batch(8, 1, d, [711, 711], [4, 2], 256), 711)


def test_time_of_sparse_pieces():
    """A merge that looks its pieces up one by one took this call from 22.6 to
    38.5 us; with tight bounds it has few pieces."""
    prefix, nodes = [711, 711], [4, 2]
    loose, tight = (U.attention_call(_batch(8, 1, 64, prefix, nodes, n), 711)[0] for n in (256, 4))
    t = U.call_times(loose, tight)
    U.log(f"[loose bounds] Nmax 256: {t[0]:.1f} us, Nmax 4: {t[1]:.1f} us")
    assert t[0] < 2.5 * t[1], t  # 3.3 one by one, 2.0 by lanes


# Plans of 6 splits (the merge for up to 8), 18 (a wave a row, every split
# requested up front) and more than 32; and, with 256-node bounds on 8 kv
# heads, plans of 4 and 20 whose partials are not requested before the lengths
# are known.
@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("Hq,Hkv,Nmax,max_prefix,lo,hi", [(8, 2, 16, 640, 2, 8), (8, 2, 16, 2200, 9, 32),
                                                          (8, 2, 31, 640, 2, 8), (8, 2, 31, 2200, 9, 32),
                                                          (8, 2, 31, 6300, 33, 64), (64, 8, 256, 6000, 2, 8),
                                                          (64, 8, 256, 40000, 9, 32)])
def test_fewer_splits_than_planned(Hq, Hkv, Nmax, max_prefix, lo, hi, d):
    """One sequence whose prefix gives 1, 2 or some of the splits that the plan
    for max_prefix allows: partials that no workgroup wrote are not used."""
    grid, units = (ltd.attn_grid(1, Nmax, Hq, Hkv, d, p, ltd.DTYPE_BF16, max_prefix + Nmax)
                   for p in (max_prefix, 1))
    assert lo <= grid // units <= hi
    for P in (0, 1, 128, 129, max_prefix // 2):
        _check(_batch(Hq, Hkv, d, [P], [13], Nmax), max_prefix)


def test_time_of_a_loose_prefix_bound():
    """A merge that requests every planned split's rows took this call from 101
    to 153 us; with max_prefix tight it takes 41."""
    b = _batch(64, 8, 128, [2225, 5070, 3000, 4000], [14, 42, 20, 30], 256, block=16)
    t = U.call_times(U.attention_call(b, 81120)[0], U.attention_call(b, 5070)[0])
    U.log(f"[loose bounds] max_prefix 81120: {t[0]:.1f} us, 5070: {t[1]:.1f} us")
    assert t[0] < 2.5 * t[1], t  # 3.7 with every planned split requested, 1.7 without


def test_time_of_sampling_with_a_loose_node_bound():
    """Workgroups without a node that first loaded the tree's links took
    acceptance over 8-node trees with Nmax 256 from 56 to 71 us."""
    B, n, voc = 4, 8, 128256
    g = torch.Generator(device="cuda")
    g.manual_seed(1)

    def call(Nmax):
        i32 = dict(dtype=torch.int32, device="cuda")
        logits = torch.randn(B, Nmax, voc, generator=g, device="cuda") * 3
        draft = torch.softmax(logits + torch.randn(B, Nmax, voc, generator=g, device="cuda"), 2)
        parents = torch.zeros(B, Nmax, **i32)
        parents[:, 0] = -1
        parents[:, 3:n] = 1
        tokens = torch.arange(Nmax, **i32).repeat(B, 1)
        nodes, uniforms = torch.full((B,), n, **i32), torch.full((B, Nmax, 2), 0.5, device="cuda")
        acc, toks, nacc = torch.zeros(B, Nmax, **i32), torch.zeros(B, Nmax, **i32), torch.zeros(B, **i32)
        ws = torch.empty(ltd.accept_sampling_workspace_size(B, Nmax, voc), dtype=torch.uint8, device="cuda")
        return lambda: ltd.tree_accept_sampling(logits, draft, tokens, parents, nodes, uniforms, acc, toks,
                                                nacc, workspace=ws)

    t = U.call_times(call(256), call(n))
    U.log(f"[loose bounds] sampling, Nmax 256: {t[0]:.1f} us, Nmax {n}: {t[1]:.1f} us")
    assert t[0] < 1.6 * t[1], t
