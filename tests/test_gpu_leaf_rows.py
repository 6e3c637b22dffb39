"""Leaf ids of outputs large enough for the two-kernel path (positions in packed order, then rows
through LDS): the sizes where its dispatch changes, tile and block remainders, every document
block width, compact packets, big trees, and more than one chunk of scratch. Ids bit for bit
against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as W
from _gpu import assert_leaves_equal, dev

pytestmark = pytest.mark.gpu

M = 1 << 20  # ids at which the path changes: 2 M from 256 trees on, 4 M from 128

# (trees, documents, features, leaves): direct below 128 trees and up to the limit, rows past it;
# trees and documents off the 64-wide tiles; 64-, 32-, 16- and 8-document blocks (136, 500, 1,200
# and 2,000 features); compact packets (700 features, 150 leaves)
CASES = [
    (127, 4 * M // 127 + 70, 20, 8), (128, 4 * M // 128, 20, 8), (128, 4 * M // 128 + 1, 20, 8),
    (255, 4 * M // 255 + 65, 20, 8), (256, 2 * M // 256, 20, 8), (256, 2 * M // 256 + 1, 20, 8),
    (257, 2 * M // 257 + 63, 136, 12), (1_000, 2_111, 136, 32), (4_099, 520, 136, 9),
    (300, 7_003, 500, 10), (300, 7_011, 1_200, 10), (300, 7_009, 2_000, 10), (300, 7_041, 700, 150),
    (2_000, 35_003, 30, 3),  # 140 MB of positions: two chunks
]


@pytest.fixture(scope="module")
def T():
    import paper_1212_2287_amd as T
    T.load_library()
    return T


@pytest.mark.parametrize("trees,docs,features,leaves", CASES)
def test_leaf_rows(T, trees, docs, features, leaves):
    import torch
    ens = W.random_ensemble(trees + docs, n_trees=trees, n_features=features, min_leaves=1, max_leaves=leaves)
    X = W.random_docs(docs, docs, features)
    flags = docs % 2
    with T.TreeEnsemble.from_ensemble(ens, flags) as m:
        x = dev(X)
        ids = m.predict_leaves(x)
        again = m.predict_leaves(x)
        torch.cuda.synchronize()
        assert torch.equal(ids, again)
        ids = ids.cpu().numpy()
    _, ref, _ = oracle.score(ens, X, rule=flags)
    assert_leaves_equal(ids, ref, f"{trees} trees x {docs} docs")


def test_leaf_rows_big_trees(T):
    import torch
    parts = [W.random_ensemble(5, 300, 60, 1, 20), W.random_ensemble(6, 1, 60, 32_768, 32_768)]
    trees = [e.tree(t) for e in parts for t in range(e.n_trees)]
    order = np.random.default_rng(1).permutation(len(trees))
    cat = [np.concatenate([trees[i][k] for i in order]) for k in range(5)]
    offs = np.concatenate([[0], np.cumsum([len(trees[i][0]) for i in order])]).astype(np.int64)
    ens = W.Ensemble(offs, *cat, 60)
    X = W.random_docs(9, 7_100, 60)
    with T.TreeEnsemble.from_ensemble(ens) as m:
        ids = m.predict_leaves(dev(X))
        torch.cuda.synchronize()
        ids = ids.cpu().numpy()
    _, ref, _ = oracle.score(ens, X)
    assert_leaves_equal(ids, ref, "big tree ids beyond 15 bits")
