"""Sampling acceptance where a node's children lie on both sides of the 64-node
words that the kernels find them in: a chain down to node first - 1, every
later node a child of the root.  The rule and its bounds are those of the
sampling parity tests."""
import pytest

import test_gpu_sampling as S
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [64, 65, 130, 256])
def test_children_across_words(n):
    rng = W.rng_for(700 + n)
    trees = []
    for first in (2, 62, 63, 64, 126, 127, 128, 191, 254):
        if first < n:
            trees.append([j - 1 if j < first else 0 for j in range(n)])
            trees[-1][0] = -1
    S._check(W.make_sampling_batch(rng, trees, 3001, temperature=1.0, draft_noise=3.0,
                                   label=f"children across words n={n}"))


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6])
def test_last_nodes(n):
    """The first nodes that no longer have one, two or three nodes after them,
    hence no such child: stars, chains and stars below a chain."""
    rng = W.rng_for(750 + n)
    trees = [W.tree_star(n), W.tree_chain(n)]
    for top in (1, 2, 3):
        if top < n:
            trees.append([j - 1 if j <= top else top for j in range(n)])
    S._check(W.make_sampling_batch(rng, trees, 3001, temperature=1.0, draft_noise=3.0,
                                   label=f"last nodes n={n}"))
