"""Which kernels a call runs, and the oracle's results from them: both sides of every rule (uniform
evaluation, terminal packets, leaf rows, ids stored directly), eager, captured and allocation-free;
every block width and both depths of the uniform kernels, terminal packets of cut trees and
partial windows, leaf rows of every block width."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as W
from _gpu import assert_leaves_equal, assert_scores_close, dev

pytestmark = pytest.mark.gpu
VALUES = np.array([-np.inf, -0.0, 0.0, 1e-42, 0.25, 0.5, 2.0, np.inf, np.nan], np.float32)
WALK, UNIFORM, TERMINAL, ROWS = 1, 2, 3, 4


@pytest.fixture(scope="module")
def T():
    import paper_1212_2287_amd as T
    T.load_library()
    assert (T.TREE_ENS_PATH_WALK, T.TREE_ENS_PATH_UNIFORM, T.TREE_ENS_PATH_TERMINAL, T.TREE_ENS_PATH_ROWS) == \
        (WALK, UNIFORM, TERMINAL, ROWS)
    return T


def _ensemble(trees, features, least, most, depth, corners):
    ens = W.random_ensemble(trees + features, trees, features, least, most, depth)
    if (ens.feature >= 0).any():
        ens.feature[np.argmax(ens.feature >= 0)] = features - 1
    if corners:  # IEEE corner values and repeats among the thresholds
        rng = np.random.default_rng(trees)
        inner = np.nonzero(ens.feature >= 0)[0]
        some = rng.choice(inner, inner.size // 10, replace=False)
        ens.threshold[some] = VALUES[:-1][rng.integers(0, len(VALUES) - 1, some.size)]
    return ens


def _docs(docs, features):
    X = W.random_docs(docs, docs, features)
    rng = np.random.default_rng(docs)
    n = docs // 10
    X[rng.integers(0, docs, n), rng.integers(0, features, n)] = VALUES[rng.integers(0, len(VALUES), n)]
    return X


# trees, features, smallest and largest tree, depth, documents, path; also what the walk takes
SCORES = [
    (1_000, 25, 1, 8, 3, 100_001, UNIFORM), (1_000, 25, 1, 8, 3, 99_999, WALK),    # 512-document blocks, split
    (1_003, 25, 1, 4, 2, 99_703, UNIFORM), (1_003, 25, 1, 4, 2, 149_552, WALK),    # 35 trees in the last chunk
    (5_761, 144, 1, 8, 3, 38_402, UNIFORM), (5_761, 144, 1, 8, 3, 34_717, WALK),   # the widest 512-document tile
    (6_441, 161, 1, 8, 3, 15_528, UNIFORM), (6_400, 160, 8, 8, 3, 15_617, WALK),   # 256-document blocks, odd rows
    (8_001, 200, 1, 4, 2, 12_801, UNIFORM), (11_600, 289, 1, 8, 3, 8_705, UNIFORM),  # whole 16-byte rows; 128
    (23_001, 575, 1, 4, 2, 4_353, UNIFORM),                                         # the widest tile of all
    (50, 1, 1, 8, 3, 2_000_003, UNIFORM), (240, 6, 1, 4, 2, 600_001, UNIFORM),      # head rounds and a split tail
    (39, 1, 8, 8, 3, 2_600_000, WALK), (2_000, 30, 9, 16, 4, 60_000, WALK),         # too few trees; too deep
    (40, 400, 150, 250, None, 62_501, TERMINAL), (40, 400, 150, 250, None, 62_499, WALK),
    (63, 767, 120, 255, None, 40_001, TERMINAL), (64, 500, 200, 200, None, 39_063, TERMINAL),
    (65, 701, 1, 512, None, 63, TERMINAL), (90, 650, 230, 400, None, 23_040, TERMINAL),  # trees beyond 255 leaves: always
    (1_535, 600, 30, 255, None, 1_000, WALK), (1_536, 600, 30, 255, None, 65, TERMINAL),
    (300, 136, 2, 32, None, 40_000, WALK),
]


@pytest.mark.parametrize("trees,features,least,most,depth,docs,path", SCORES)
def test_score_paths(T, trees, features, least, most, depth, docs, path):
    import torch
    flags, bags = docs % 2, 1 + docs % 3
    ens = _ensemble(trees, features, least, most, depth, True)
    X = _docs(docs, features)
    with T.TreeEnsemble.from_arrays(ens.tree_offsets, ens.feature, ens.threshold, ens.left, ens.right, ens.value, flags,
                                    1, bags) as m:
        assert m.last_path() == T.TREE_ENS_PATH_NONE
        x = dev(X)
        s = m.predict(x)
        assert m.last_path() == path
        again = m.predict(x)
        out = torch.empty_like(s)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            m.predict(x, out)
        assert m.last_path() == path
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(s, again) and torch.equal(s, out)
        if docs * features * 2 <= 14 << 20:  # room for the split sums too
            free = m.predict_noalloc(x, torch.empty_like(s))
            assert m.last_path() == path
            assert torch.equal(s, free)
        elif path == UNIFORM:
            free = m.predict_noalloc(x, torch.empty_like(s))
            assert m.last_path() == (UNIFORM if docs * features * 2 <= 16 << 20 else WALK)
            out = free
        s, out = s.cpu().numpy(), out.cpu().numpy()
    ref, _, _ = oracle.score(ens, X, rule=flags)
    assert_scores_close(s, ref / bags, "eager")
    assert_scores_close(out, ref / bags, "allocation-free")


M = 1 << 20


@pytest.mark.parametrize("trees,features,leaves,docs,path", [
    (127, 20, 8, 4 * M // 127 + 70, WALK), (128, 20, 8, 4 * M // 128, WALK), (128, 20, 8, 4 * M // 128 + 1, ROWS),
    (255, 20, 8, 4 * M // 255 + 65, ROWS), (256, 20, 8, 2 * M // 256, WALK), (256, 20, 8, 2 * M // 256 + 1, ROWS),
    (300, 500, 10, 7_003, ROWS), (300, 1_200, 10, 7_011, ROWS), (511, 2_000, 10, 6_009, WALK), (513, 2_000, 10, 5_007, ROWS),
    (300, 700, 150, 7_041, ROWS), (2_000, 30, 3, 70_003, ROWS),
])
def test_leaf_id_paths(T, trees, features, leaves, docs, path):
    import torch
    flags = docs % 2
    ens = _ensemble(trees, features, 1, leaves, None, False)
    X = _docs(docs, features)
    with T.TreeEnsemble.from_ensemble(ens, flags) as m:
        x = dev(X)
        ids = m.predict_leaves(x)
        assert m.last_path() == path
        out = torch.empty_like(ids)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            m.predict_leaves(x, out)
        assert m.last_path() == WALK  # captured: stored directly
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(ids, out)
        ids = ids.cpu().numpy()
    assert_leaves_equal(ids, oracle.score(ens, X, rule=flags)[1], f"{trees} trees x {docs} documents")


@pytest.mark.parametrize("trees,features,leaves,n_out,docs,path", [
    (17, 20, 8, 8, 4_095, WALK), (17, 20, 8, 8, 4_097, ROWS), (17, 20, 8, 4, 5_000, WALK), (1, 20, 1, 9, 5_000, ROWS),
    (1_100, 20, 8, 5, 4_399, WALK), (1_100, 20, 8, 5, 4_400, ROWS), (1_100, 20, 8, 33, 5_499, WALK),
    (1_100, 20, 8, 33, 5_500, ROWS), (4_097, 5, 3, 5, 16_400, WALK), (2_100, 5, 3, 5, 32_768, ROWS),
    (2_100, 5, 3, 5, 32_769, WALK), (60, 500, 10, 16, 5_002, ROWS), (60, 1_200, 10, 13, 5_003, ROWS),
    (60, 2_000, 10, 6, 5_001, ROWS), (70, 700, 150, 7, 5_005, ROWS),
])
def test_leaf_vector_paths(T, trees, features, leaves, n_out, docs, path):
    import torch
    ens = _ensemble(trees, features, 1, leaves, None, False)
    vals = W.make_leaf_vectors(ens, n_out, "dense", seed=docs)
    X = _docs(docs, features)
    with T.TreeEnsemble.from_ensemble(ens, leaf_values=vals, n_bags=2) as m:
        x = dev(X)
        got = m.predict(x)
        assert m.last_path() == path
        out = torch.empty_like(got)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            m.predict(x, out)
        assert m.last_path() == path
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, out)
        if docs * (trees + (features if features >= 700 else 0)) * 2 <= 14 << 20:
            free = m.predict_noalloc(x, torch.empty_like(got))
            assert m.last_path() == path
            assert torch.equal(got, free)
        got = got.cpu().numpy()
    ref = oracle.score_multi(ens, vals, X, n_bags=2)
    for c in range(n_out):
        assert_scores_close(got[:, c], ref[:, c], f"output {c}")


@pytest.mark.parametrize("trees,features,least,most,depth,docs,n_out,path", [
    (1_000, 25, 1, 8, 3, 100_001, 1, UNIFORM), (1_003, 25, 1, 4, 2, 99_703, 1, UNIFORM),
    (90, 650, 230, 400, None, 20_001, 1, TERMINAL), (300, 20, 1, 8, None, 5_001, 6, ROWS), (300, 20, 1, 8, None, 2_001, 6, WALK),
])
def test_leaf_values_that_are_not_finite(T, trees, features, least, most, depth, docs, n_out, path):
    """Infinities and NaN among the leaves: each document's score is that of the leaves it reaches, whatever the
    padding, the cut trees' other pieces and the split sums hold."""
    import torch
    ens = _ensemble(trees, features, least, most, depth, False)
    vals = W.make_leaf_vectors(ens, n_out, "dense", seed=docs) if n_out > 1 else ens.value.reshape(-1, 1)
    rng = np.random.default_rng(docs)
    leaves = np.setdiff1d(np.nonzero(ens.feature < 0)[0], ens.tree_offsets[:-1])  # not a whole tree
    rows = rng.choice(leaves, 6, replace=False)
    for c in range(n_out):
        vals[rows, c] = np.array([np.inf, -np.inf, np.nan], np.float32)[(np.arange(6) + c) % 3]
    X = W.random_docs(docs, docs, features)
    with T.TreeEnsemble.from_ensemble(ens, leaf_values=vals if n_out > 1 else None) as m:
        got = m.predict(dev(X))
        assert m.last_path() == path
        torch.cuda.synchronize()
        got = got.cpu().numpy().reshape(docs, n_out)
    with np.errstate(invalid="ignore"):
        ref = (oracle.score_multi(ens, vals, X) if n_out > 1 else oracle.score(ens, X)[0].reshape(-1, 1)).astype(np.float32)
    assert (~np.isfinite(ref)).any() and np.isfinite(ref).any()
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref))
    assert np.array_equal(np.isneginf(got), np.isneginf(ref))
    for c in range(n_out):
        f = np.isfinite(ref[:, c])
        assert_scores_close(got[f, c], ref[f, c], f"output {c}")
