"""Coded models of one output on the GPU against the oracle, most of them by terminal packets
(test_gpu_routes.py asserts which): tree sizes on both sides of a window, cut trees, the widest document
tile, partial groups and blocks, split batches, both tie rules, IEEE corner values, bags."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as W
from _gpu import assert_scores_close, dev

pytestmark = pytest.mark.gpu
VALUES = np.array([-np.inf, -0.0, 0.0, 1e-42, 0.25, 0.5, 2.0, np.inf, np.nan], np.float32)


@pytest.fixture(scope="module")
def T():
    import paper_1212_2287_amd as T
    T.load_library()
    return T


def _check(T, ens, X, flags, bags, what):
    import torch
    with T.TreeEnsemble.from_arrays(ens.tree_offsets, ens.feature, ens.threshold, ens.left, ens.right, ens.value, flags,
                                    1, bags) as m:
        x = dev(X)
        s = m.predict(x)
        again = m.predict(x)
        torch.cuda.synchronize()
        assert torch.equal(s, again)
        s = s.cpu().numpy()
    ref, _, _ = oracle.score(ens, X, rule=flags)
    assert_scores_close(s, ref / bags, what)


# trees, smallest and largest tree (leaves), features, documents, bags; models whose mean tree is large
# enough for coded documents
@pytest.mark.parametrize("trees,least,most,features,docs,bags", [
    (40, 150, 250, 400, 50_001, 1), (63, 120, 260, 767, 33_000, 2), (64, 200, 200, 500, 31_300, 1),
    (65, 1, 512, 701, 31_000, 3), (257, 200, 300, 700, 17_003, 1), (90, 230, 270, 766, 23_000, 1),
    (90, 230, 400, 650, 23_040, 1), (1_100, 100, 260, 600, 2_049, 1),
])
def test_term_scores(T, trees, least, most, features, docs, bags):
    flags = docs % 2
    ens = W.random_ensemble(trees + docs, trees, features, least, most)
    ens.feature[np.argmax(ens.feature >= 0)] = features - 1 if (ens.feature >= 0).any() else -1
    rng = np.random.default_rng(docs)
    inner = np.nonzero(ens.feature >= 0)[0]
    some = rng.choice(inner, inner.size // 8, replace=False)
    ens.threshold[some] = VALUES[:-1][rng.integers(0, len(VALUES) - 1, some.size)]
    X = W.random_docs(docs, docs, features)
    X[rng.integers(0, docs, docs), rng.integers(0, features, docs)] = VALUES[rng.integers(0, len(VALUES), docs)]
    _check(T, ens, X, flags, bags, f"{trees} trees of {least}-{most} leaves, {features} features")


@pytest.mark.parametrize("docs", [1, 64, 65, 640, 2_000, 16_384, 16_449, 40_000])
def test_term_batches(T, docs):
    ens = W.random_ensemble(5, 1_024, 450, 100, 260)
    _check(T, ens, W.random_docs(docs, docs, 450), 0, 1, f"{docs} documents")
