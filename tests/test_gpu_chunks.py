"""Batches of shallow models whose threshold codes exceed a chunk's memory: taken in chunks of whole
rounds, with the oracle's scores around the boundary, those of smaller calls everywhere, and no more
device memory than a chunk needs."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as W
from _gpu import assert_scores_close

pytestmark = pytest.mark.gpu
CHUNK = 256 << 20


@pytest.fixture(scope="module")
def T():
    import paper_1212_2287_amd as T
    T.load_library()
    return T


# trees, features, depth, documents of a block, documents past the first chunk
@pytest.mark.parametrize("trees,features,depth,block,past", [
    (1_000, 25, 2, 512, 1), (1_000, 25, 2, 512, 2_500_007), (2_320, 58, 3, 512, 1_400_000), (6_400, 160, 3, 256, 400_001),
])
def test_chunks(T, trees, features, depth, block, past):
    import torch
    round_docs = block * 256
    chunk = CHUNK // (round_docs * features * 2) * round_docs
    docs = chunk + past
    ens = W.random_ensemble(trees, trees, features, 1 << depth, 1 << depth, depth)
    ens.feature[np.argmax(ens.feature >= 0)] = features - 1
    gen = torch.Generator(device="cuda").manual_seed(docs)
    x = torch.rand((docs, features), device="cuda", generator=gen)
    out = torch.full((docs + 64,), -1.0, device="cuda")
    torch.cuda.synchronize()
    with T.TreeEnsemble.from_ensemble(ens) as m:
        m.predict(x[:1_000].contiguous())
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        free = torch.cuda.mem_get_info()[0]
        m.predict(x, out[:docs])
        torch.cuda.synchronize()
        took = free - torch.cuda.mem_get_info()[0]
        assert took <= CHUNK + (16 << 20), f"{took >> 20} MiB"
        assert (out[docs:] == -1.0).all()
        for lo in range(0, docs, 500_000):  # smaller calls
            part = m.predict(x[lo:lo + 500_000])
            assert torch.allclose(out[lo:lo + part.numel()], part, rtol=1e-5, atol=1e-6), lo
        torch.cuda.synchronize()
    for lo, hi in ((0, 300), (chunk - 600, min(chunk + 600, docs)), (docs - 200, docs)):
        ref, _, _ = oracle.score(ens, x[lo:hi].cpu().numpy())
        assert_scores_close(out[lo:hi].cpu().numpy(), ref, f"documents {lo} to {hi}")
