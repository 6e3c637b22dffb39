"""The launch planner on packed models: shapes a launch can run, for batches and models of all kinds; no
split without something to gain; shapes that were measured: the ones picked are the fastest of
their batch, or within a few percent; and the choice of kernels on both sides of each rule."""
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
    for fn in (lib.plan_model, lib.plan_rules):
        fn.argtypes = [ctypes.c_int32, P, P, P, P, P, P, ctypes.c_int32, ctypes.c_int32, P, P, P]
    return lib


def _model(ens, n_out):
    arrs = [np.ascontiguousarray(a, t) for a, t in ((ens.tree_offsets, np.int64), (ens.feature, np.int32),
            (ens.threshold, np.float32), (ens.left, np.int32), (ens.right, np.int32), (ens.value, np.float32))]
    if n_out > 1:
        arrs[5] = np.zeros((ens.n_nodes, n_out), np.float32)
    return arrs, (ens.n_trees, *[a.ctypes.data for a in arrs], n_out)


def _plan(lib, ens, asks, n_out=1):
    """(level, head, splits, tiles, blocks) of each (work, documents)."""
    _keep, args = _model(ens, n_out)
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


def _forest(trees, features, least, most, depth=None):
    """`trees` trees, at most 64 different ones; the widest feature is read."""
    base = W.random_ensemble(features + trees + least, min(trees, 64), features, least, most, depth, thr_values=VALUES)
    base.feature[np.argmax(base.feature >= 0)] = features - 1
    each = [base.tree(t % base.n_trees) for t in range(trees)]
    offsets = np.concatenate([[0], np.cumsum([len(t[0]) for t in each])]).astype(np.int64)
    return W.Ensemble(offsets, *[np.concatenate([t[k] for t in each]) for k in range(5)], features)


@pytest.mark.parametrize("trees,features,least,most,work,docs,shapes", [
    # leaf ids reduce nothing: 8.5 us in two shares, 11.6 whole
    (128, 136, 32, 32, POSITIONS, 100, [(0, 2)]), (128, 136, 32, 32, POSITIONS, 3_000, [(0, 2)]),
    # 32-document blocks: 124 us whole, 140 with 170 blocks in three
    (1_000, 700, 64, 64, SCORES, 30_011, [(0, 1)]),
    # tiles of up to 6 rounds, 1.25 on average: 22.7 us in 9 shares, 28.3 in 32
    (600, 136, 5, 300, SCORES, 3_000, [(0, s) for s in range(5, 13)]),
    # terminal packets, 105 blocks: 187 us in halves, 234 in seven shares
    (5_000, 700, 256, 256, TERMINAL, 6_700, [(0, 2)]), (1_000, 700, 512, 512, TERMINAL, 6_700, [(0, 2)]),
    # 80 packets, 8 blocks: 51.3 us in 32 shares of 2 or 3, 58.9 in 27
    (5_000, 700, 256, 256, TERMINAL, 500, [(0, 32)]),
    # leaf vectors, 256 blocks: 121 us in halves, 135 whole; 45.2 whole, 47.7 in halves
    (4_096, 136, 16, 16, VECTOR, 16_383, [(0, 2)]), (1_000, 136, 32, 32, VECTOR, 16_383, [(0, 1)]),
    # 300 trees, 63 blocks of 8 documents: 13.5 us whole, 15.7 in three shares
    (300, 2_000, 30, 30, SCORES, 500, [(0, 1)]),
])
def test_measured_shapes(lib, trees, features, least, most, work, docs, shapes):
    ens = _forest(trees, features, least, most)
    _, head, splits, _, _ = _plan(lib, ens, [(work, docs)], 4 if work == VECTOR else 1)[0]
    assert (head, splits) in shapes or (splits == 1 and (0, 1) in shapes)


def _pays(lib, ens, rule, docs, n_out=1):
    _keep, args = _model(ens, n_out)
    n = len(docs)
    pays = np.zeros(n, np.int32)
    assert lib.plan_rules(*args, n, np.full(n, rule, np.int32).ctypes.data, np.array(docs, np.int64).ctypes.data,
                          pays.ctypes.data) == 0
    return pays.tolist()


@pytest.mark.parametrize("trees,features,least,most,walked,terminal", [
    # documents at which the walk by compact packets was the faster, and the terminal packets
    (1_024, 700, 256, 256, [500, 1_000, 2_000], [3_500, 6_700, 20_000]),
    (300, 450, 200, 200, [100, 2_000, 6_700], [10_000, 20_000]),
    (1_100, 450, 100, 255, [1_000, 2_000], [6_700, 50_000]),
    (2_000, 600, 150, 150, [], [1, 64, 1_000, 50_000]),
    (60, 600, 400, 600, [], [1, 1_000]),           # trees beyond the compact packets
    (1_000, 136, 32, 32, [100, 100_000], []),      # float documents
])
def test_terminal_packets_where_they_pay(lib, trees, features, least, most, walked, terminal):
    ens = _forest(trees, features, least, most)
    assert _pays(lib, ens, 1, walked) == [0] * len(walked)
    assert _pays(lib, ens, 1, terminal) == [1] * len(terminal)


@pytest.mark.parametrize("trees,features,leaves,outputs,walked,rows", [
    (1_000, 136, 32, 8, [500, 2_000], [6_000, 16_384, 200_000]), (1_000, 136, 32, 64, [2_000, 4_096], [6_000, 50_000]),
    (4_000, 30, 8, 6, [4_096, 8_192, 33_000, 50_000, 200_000], [16_384, 32_000]),  # walks cheaper than gathers
    (4_000, 30, 8, 16, [8_192, 50_000], [16_384]), (3_000, 30, 8, 6, [50_000], [16_384]),
    (3_000, 30, 8, 12, [6_000], [16_384, 50_000]), (2_000, 30, 8, 6, [6_000], [12_000, 16_384, 50_000]),
    (10, 20, 8, 5, [], [4_096, 200_000]), (4_096, 136, 16, 24, [8_192], [16_384, 100_000]),
    (6_000, 30, 8, 8, [4_096, 50_000], []),     # chunks too small
    (300, 1_200, 10, 10, [], [4_096, 200_000]), (300, 136, 32, 4, [4_096, 50_000], []),
])
def test_leaf_rows_where_they_pay(lib, trees, features, leaves, outputs, walked, rows):
    ens = _forest(trees, features, leaves, leaves)
    assert _pays(lib, ens, 3, walked, outputs) == [0] * len(walked)
    assert _pays(lib, ens, 3, rows, outputs) == [1] * len(rows)


@pytest.mark.parametrize("trees,features,depth,walked,uniform", [
    # documents; 512-, 256- and 128-document blocks
    (1_000, 25, 2, [50_000, 140_000], [100_000, 450_000, 2_500_000]), (1_000, 25, 3, [50_000], [100_000, 300_000, 1_200_000]),
    (5_440, 136, 2, [18_382, 36_764, 82_720], [128_676, 459_558]), (5_440, 136, 3, [9_191, 18_382], [128_676, 459_558]),
    (20_000, 136, 3, [2_500], [10_000, 60_000, 1_000_000]), (8_000, 200, 3, [2_500], [12_500, 87_500, 312_500]),
    (12_000, 300, 3, [16_666, 25_000], [100_000, 208_333]), (16_800, 420, 3, [8_333, 11_904, 17_857], [71_428]),
    (3_000, 136, 3, [33_333, 400_000], []),  # too few trees for their columns
    (2_000, 30, 4, [100_000], []),           # deeper trees
])
def test_uniform_evaluation_where_it_pays(lib, trees, features, depth, walked, uniform):
    ens = _forest(trees, features, 1 << depth, 1 << depth, depth)
    assert _pays(lib, ens, 0, walked) == [0] * len(walked)
    assert _pays(lib, ens, 0, uniform) == [1] * len(uniform)


@pytest.mark.parametrize("trees,features,leaves,direct,rows", [
    (127, 20, 8, [1_000_000], []), (128, 136, 32, [24_576, 32_768], [32_769, 327_680]),
    (256, 136, 32, [8_192], [8_193, 163_840]), (1_000, 136, 32, [1_048, 2_097], [2_098, 41_943]),
    (300, 500, 10, [6_990], [6_991]), (300, 1_200, 10, [6_990], [6_991]),          # 32 and 16 documents a block
    (300, 2_600, 30, [6_990, 139_810], []), (511, 2_000, 10, [100_000], []), (512, 2_000, 10, [4_096], [4_097]),  # 8
])
def test_ids_stored_directly(lib, trees, features, leaves, direct, rows):
    ens = _forest(trees, features, leaves, leaves)
    assert _pays(lib, ens, 2, direct) == [1] * len(direct)
    assert _pays(lib, ens, 2, rows) == [0] * len(rows)
