"""Attention calls whose bounds (Nmax, max_prefix) are far above their data, as
a decoder makes them whose buffers are sized once: results against the oracle,
with a workspace full of NaN so that a partial nobody wrote shows, and the
time against the same call with tight bounds."""
import numpy as np
import pytest
import torch

import gpu_util as U
import oracle
import paper_2603_01639_amd as ltd
import workloads as W

pytestmark = pytest.mark.gpu


def _batch(Hq, Hkv, d, prefix, nodes, Nmax, block=0):
    rng = np.random.default_rng(sum(prefix) * 31 + sum(nodes))
    trees = [W.tree_uniform_parent(rng, n) for n in nodes]
    return W.make_batch(rng, dtype=W.DTYPE_BF16, Hq=Hq, Hkv=Hkv, d=d, prefix=prefix, trees=trees,
                        tokens=[W.distinct_sibling_tokens(rng, t, 500) for t in trees], Voc=500, p_match=0.7,
                        Nmax=Nmax, block_size=block, label=f"d={d} P={prefix} N={nodes} Nmax={Nmax}")


def _call(b, max_prefix):
    """The call on device copies, its output and a workspace of NaN."""
    dev = U.upload(b)
    out = torch.zeros(tuple(b.q.shape), dtype=torch.bfloat16, device="cuda")
    size = ltd.attn_workspace_size(b.B, b.Nmax, b.Hq, b.Hkv, b.d, max_prefix, b.dtype)
    ws = torch.full((max(size, 1),), 0xFF, dtype=torch.uint8, device="cuda")

    def run():
        ltd.tree_verify_attn(dev.q, dev.k, dev.v, dev.prefix_len, dev.parents, dev.n_nodes, out,
                             max_prefix=max_prefix, block_table=dev.block_table, num_blocks=b.num_blocks,
                             workspace=ws)
    return run, out


def _check(b, max_prefix):
    U.log(f"[loose bounds] {b.label} max_prefix={max_prefix}")
    run, out = _call(b, max_prefix)
    run()
    U.compare_attention(b, U.to_host(out), U.oracle_attention(b))


def _times(*calls, n=10, rounds=7):
    """Fastest time of each call in us, in graphs of n replayed in turn."""
    graphs = []
    for run in calls:
        run()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for _ in range(n):
                run()
        g.replay()
        graphs.append(g)
    best = [float("inf")] * len(calls)
    for _ in range(rounds):
        for i, g in enumerate(graphs):
            a, z = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            g.replay()
            z.record()
            z.synchronize()
            best[i] = min(best[i], a.elapsed_time(z) * 1e3 / n)
    return best


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
    loose, tight = (_call(_batch(8, 1, 64, prefix, nodes, n), 711)[0] for n in (256, 4))
    t = _times(loose, tight)
    U.log(f"[loose bounds] Nmax 256: {t[0]:.1f} us, Nmax 4: {t[1]:.1f} us")
    assert t[0] < 2.5 * t[1], t  # 3.3 one by one, 2.0 by lanes
