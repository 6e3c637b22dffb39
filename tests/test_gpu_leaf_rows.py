"""Leaf ids (and sums of leaf vectors, below) of outputs large enough for the two-kernel path (positions in packed order, then rows
through LDS): the sizes where its dispatch changes, tile and block remainders, every document
block width, compact packets, big trees, and more than one chunk of scratch. Ids bit for bit,
sums within the score tolerance, against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as W
from _gpu import assert_leaves_equal, assert_scores_close, dev

pytestmark = pytest.mark.gpu

M = 1 << 20  # ids at which the path changes: 2 M from 256 trees on, 4 M from 128

# (trees, documents, features, leaves): direct below 128 trees and up to the limit, rows past it;
# trees and documents off the 64-wide tiles; 64-, 32-, 16- and 8-document blocks (136, 500, 1,200
# and 2,000 features; the last stored directly: fewer than 512 trees); compact packets (700 features, 150 leaves)
CASES = [
    (127, 4 * M // 127 + 70, 20, 8), (128, 4 * M // 128, 20, 8), (128, 4 * M // 128 + 1, 20, 8),
    (255, 4 * M // 255 + 65, 20, 8), (256, 2 * M // 256, 20, 8), (256, 2 * M // 256 + 1, 20, 8),
    (257, 2 * M // 257 + 63, 136, 12), (1_000, 2_111, 136, 32), (4_099, 520, 136, 9),
    (300, 7_003, 500, 10), (300, 7_011, 1_200, 10), (300, 7_009, 2_000, 10), (300, 7_041, 700, 150),
    (2_000, 70_003, 30, 3),  # 280 MB of positions: two chunks
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


@pytest.mark.parametrize("trees,docs,features,leaves,n_out", [
    (3, 4_095, 20, 8, 5), (3, 4_096, 20, 8, 5), (17, 4_097, 20, 8, 8),  # the size where the path changes
    (1, 5_000, 20, 1, 9),          # fewer trees than waves; a lone leaf; an odd last group of outputs
    (4_097, 16_400, 5, 3, 5),      # one tree too many for the chunks: one walk per four outputs
    (4_096, 33_001, 5, 3, 5),      # two chunks, the second short
    (3_000, 12_007, 30, 40, 12),   # more than 65,536 rows: the stored 16 bits wrap within trees
    (60, 5_003, 1_200, 10, 13), (60, 5_001, 2_000, 10, 6), (60, 5_002, 500, 10, 16), (70, 5_005, 700, 150, 7),
])
def test_vector_rows(T, trees, docs, features, leaves, n_out):
    import torch
    ens = W.random_ensemble(trees + docs, trees, features, 1, leaves)
    X = W.random_docs(docs, docs, features)
    vals = W.make_leaf_vectors(ens, n_out, "dense", seed=docs)
    with T.TreeEnsemble.from_ensemble(ens, leaf_values=vals, n_bags=2) as m:
        x = dev(X)
        got = m.predict(x)
        again = m.predict(x)
        torch.cuda.synchronize()
        assert torch.equal(got, again)
        got = got.cpu().numpy()
    ref = oracle.score_multi(ens, vals, X, n_bags=2)
    for c in range(n_out):
        assert_scores_close(got[:, c], ref[:, c], f"output {c}")


def test_vector_rows_big_tree(T):
    parts = [W.random_ensemble(5, 30, 60, 1, 20), W.random_ensemble(6, 3, 60, 32_768, 32_768)]
    trees = [e.tree(t) for e in parts for t in range(e.n_trees)]
    cat = [np.concatenate([t[k] for t in trees]) for k in range(5)]
    offs = np.concatenate([[0], np.cumsum([len(t[0]) for t in trees])]).astype(np.int64)
    ens = W.Ensemble(offs, *cat, 60)
    X = W.random_docs(9, 4_200, 60)
    vals = W.make_leaf_vectors(ens, 6, "dense", seed=1)
    with T.TreeEnsemble.from_ensemble(ens, leaf_values=vals) as m:
        got = m.predict(dev(X)).cpu().numpy()
    ref = oracle.score_multi(ens, vals, X)
    for c in range(6):
        assert_scores_close(got[:, c], ref[:, c], f"output {c}")
