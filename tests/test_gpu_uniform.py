"""Shallow models on the GPU against the oracle, in sizes of 40 trees per feature and 1e8 walks, scored by
uniform evaluation or the walk (test_gpu_routes.py asserts which): every width of the document tile,
both depths, partial blocks and chunks, whole rounds of blocks with a split tail, batches split over
their trees, both tie rules, bags, allocation-free calls, and batches too small for it."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as W
from _gpu import assert_scores_close, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    import paper_1212_2287_amd as T
    T.load_library()
    return T


# depth, trees, features, documents
@pytest.mark.parametrize("depth,trees,features,docs,bags", [
    (3, 1_000, 25, 100_001, 1),   # 512-document blocks, split over the trees
    (3, 5_761, 144, 17_921, 3),   # the widest 512-document tile; rows of whole 16 bytes; 35 blocks + 1 doc
    (3, 5_801, 145, 17_300, 1),   # 256-document blocks, odd rows
    (3, 11_600, 289, 8_705, 1),   # 128-document blocks
    (3, 50, 1, 2_000_003, 1),     # one column; head rounds and a split tail
    (2, 1_003, 25, 140_000, 1),
    (2, 240, 6, 600_001, 2),
])
def test_uniform_scores(T, depth, trees, features, docs, bags):
    import torch
    flags = docs % 2
    values = np.array([-np.inf, -0.0, 0.0, 1e-42, 0.5, 2.0, np.inf, np.nan], np.float32)
    ens = W.random_ensemble(trees + docs, trees, features, 1, 1 << depth, depth)
    rng = np.random.default_rng(docs)
    inner = np.nonzero(ens.feature >= 0)[0]
    some = rng.choice(inner, inner.size // 10, replace=False)  # ties and corner values among the thresholds
    ens.threshold[some] = values[:-1][rng.integers(0, len(values) - 1, some.size)]
    X = W.random_docs(docs, docs, features)
    X[rng.integers(0, docs, docs // 10), rng.integers(0, features, docs // 10)] = values[rng.integers(0, len(values), docs // 10)]
    with T.TreeEnsemble.from_arrays(ens.tree_offsets, ens.feature, ens.threshold, ens.left, ens.right, ens.value, flags,
                                    1, bags) as m:
        x = dev(X)
        s = m.predict(x)
        again = m.predict(x)
        walked = m.predict_noalloc(x, torch.empty_like(s))  # the same kernels, while their scratch fits 16 MiB
        few = m.predict(x[:700].contiguous())               # too small a batch: the walk
        torch.cuda.synchronize()
        assert torch.equal(s, again)
        s, walked, few = s.cpu().numpy(), walked.cpu().numpy(), few.cpu().numpy()
    ref, _, _ = oracle.score(ens, X, rule=flags)
    assert_scores_close(s, ref / bags, "uniform")
    assert_scores_close(walked, ref / bags, "allocation-free")
    assert_scores_close(few, ref[:700] / bags, "walk, small batch")


def test_uniform_two_streams_and_capture(T):
    import torch
    ens = W.random_ensemble(3, 2_000, 30, 8, 8, 3)
    X = W.random_docs(5, 60_000, 30)
    ref, _, _ = oracle.score(ens, X)
    with T.TreeEnsemble.from_ensemble(ens) as m:
        x = dev(X)
        outs = []
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        torch.cuda.synchronize()
        for i in range(6):
            with torch.cuda.stream(streams[i % 2]):
                outs.append(m.predict(x))
        torch.cuda.synchronize()
        for o in outs:
            assert torch.equal(o, outs[0])
        assert_scores_close(outs[0].cpu().numpy(), ref, "eager on two streams")
        out = torch.zeros(60_000, device="cuda")
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            m.predict(x, out)
        for _ in range(3):
            out.zero_()
            g.replay()
            eager = m.predict(x)
            torch.cuda.synchronize()
            assert_scores_close(out.cpu().numpy(), ref, "replay")
            assert torch.equal(eager, outs[0])
