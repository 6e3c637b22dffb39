"""The launch planner on packed models: shapes a launch can run, for batches and models of all kinds; no
split without something to gain; and shapes that were measured: the ones picked are the fastest of
their batch, or within a few percent."""
from __future__ import annotations

import ctypes
import os
import subprocess

import numpy as np
import pytest

import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1212_2287_amd", "csrc")
SCORES, VECTOR, POSITIONS, TERMINAL = range(4)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("plan") / "libplan.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, os.path.join(ROOT, "tests", "plan_emu.cpp"),
                    os.path.join(CSRC, "pack.cpp"), "-o", out], check=True)
    lib = ctypes.CDLL(out)
    P = ctypes.c_void_p
    lib.plan_model.argtypes = [ctypes.c_int32, P, P, P, P, P, P, ctypes.c_int32, ctypes.c_int32, P, P, P]
    return lib


def _plan(lib, ens, asks, n_out=1):
    """(level, head, splits, tiles) of each (work, documents)."""
    arrs = [np.ascontiguousarray(a, t) for a, t in ((ens.tree_offsets, np.int64), (ens.feature, np.int32),
            (ens.threshold, np.float32), (ens.left, np.int32), (ens.right, np.int32), (ens.value, np.float32))]
    if n_out > 1:
        arrs[5] = np.zeros((ens.n_nodes, n_out), np.float32)
    args = (ens.n_trees, *[a.ctypes.data for a in arrs], n_out)
    out = np.zeros((len(asks), 5), np.int64)
    work = np.array([w for w, _ in asks], np.int32)
    one = np.ones(len(asks), np.int64)
    assert lib.plan_model(*args, len(asks), work.ctypes.data, one.ctypes.data, out.ctypes.data) == 0
    docs = np.array([64 if w == TERMINAL else out[i, 4] for i, (w, _) in enumerate(asks)])
    blocks = (np.array([d for _, d in asks], np.int64) + docs - 1) // docs
    assert lib.plan_model(*args, len(asks), work.ctypes.data, blocks.ctypes.data, out.ctypes.data) == 0
    return [tuple(int(v) for v in o[:4]) + (int(b),) for o, b in zip(out, blocks)]


VALUES = np.sort(np.random.default_rng(7).random(200, dtype=np.float32))


@pytest.mark.parametrize("trees,features,least,most", [
    (10, 136, 8, 8), (300, 46, 2, 200), (600, 136, 5, 300), (300, 1_200, 10, 10), (300, 2_000, 30, 30), (1, 5, 1, 1),
    (500, 300, 30, 30), (400, 700, 64, 64), (200, 700, 256, 256), (60, 600, 400, 600), (2, 136, 5_000, 5_000),
])
def test_shapes_can_be_launched(lib, trees, features, least, most):
    ens = W.random_ensemble(trees + features, trees, features, least, most, thr_values=VALUES)
    docs = sorted({int(v) for v in np.geomspace(1, 2e6, 60)})
    for work in (SCORES, VECTOR, POSITIONS, TERMINAL):
        for level, head, splits, tiles, blocks in _plan(lib, ens, [(work, d) for d in docs], 3 if work == VECTOR else 1):
            assert splits >= 1 and 0 <= head
            if splits > 1:
                assert splits <= tiles and head < blocks and (head == 0 or level == 0)
            assert head <= blocks


@pytest.mark.parametrize("trees,features,least,most,work,docs,shapes", [
    # leaf ids reduce nothing: 8.5 us in two shares, 11.6 whole
    (128, 136, 32, 32, POSITIONS, 100, [(0, 2)]), (128, 136, 32, 32, POSITIONS, 3_000, [(0, 2)]),
    # 32-document blocks: 124 us whole, 140 with 170 blocks in three
    (1_000, 700, 64, 64, SCORES, 30_011, [(0, 1)]),
    # tiles of up to 6 rounds, 1.25 on average: 22.7 us in 9 shares, 28.3 in 32
    (600, 136, 5, 300, SCORES, 3_000, [(0, s) for s in range(5, 13)]),
    # terminal packets, 105 blocks: 187 us in halves, 234 in seven shares
    (5_000, 700, 256, 256, TERMINAL, 6_700, [(0, 2)]), (1_000, 700, 512, 512, TERMINAL, 6_700, [(0, 2)]),
    # 300 trees, 63 blocks of 8 documents: 13.5 us whole, 15.7 in three shares
    (300, 2_000, 30, 30, SCORES, 500, [(0, 1)]),
])
def test_measured_shapes(lib, trees, features, least, most, work, docs, shapes):
    base = W.random_ensemble(features + trees + least, min(trees, 64), features, least, most, thr_values=VALUES)
    each = [base.tree(t % base.n_trees) for t in range(trees)]
    offsets = np.concatenate([[0], np.cumsum([len(t[0]) for t in each])]).astype(np.int64)
    ens = W.Ensemble(offsets, *[np.concatenate([t[k] for t in each]) for k in range(5)], features)
    _, head, splits, _, _ = _plan(lib, ens, [(work, docs)])[0]
    assert (head, splits) in shapes or (splits == 1 and (0, 1) in shapes)
