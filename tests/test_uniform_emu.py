"""Tables of uniform evaluation (shallow trees), evaluated on the host in the kernel's arithmetic and
compared with the oracle: which models take them, both depths, uneven and single-leaf trees, both tie
rules, IEEE corner values, repeated thresholds, and every width of the document tile."""
from __future__ import annotations

import ctypes
import os
import subprocess

import numpy as np
import pytest

import oracle
import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1212_2287_amd", "csrc")
VALUES = np.array([-np.inf, -1.5, -0.0, 0.0, 1e-42, 0.25, 0.5, 3.0, 1e30, np.inf], np.float32)


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("emu") / "libpackemu.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC,
                    os.path.join(ROOT, "tests", "pack_emu.cpp"), os.path.join(CSRC, "pack.cpp"), "-o", out], check=True)
    lib = ctypes.CDLL(out)
    P = ctypes.c_void_p
    lib.emu_uniform.argtypes = [ctypes.c_int32, P, P, P, P, P, P, ctypes.c_uint32, P, ctypes.c_int64, ctypes.c_int32, P, P]
    lib.emu_message.restype = ctypes.c_char_p
    return lib


def _uniform(lib, ens, X, flags):
    arrs = [np.ascontiguousarray(a, t) for a, t in ((ens.tree_offsets, np.int64), (ens.feature, np.int32),
            (ens.threshold, np.float32), (ens.left, np.int32), (ens.right, np.int32), (ens.value, np.float32))]
    scores, plan = np.empty(X.shape[0]), np.zeros(3, np.int32)
    rc = lib.emu_uniform(ens.n_trees, *[a.ctypes.data for a in arrs], flags, X.ctypes.data, X.shape[0], X.shape[1],
                         scores.ctypes.data, plan.ctypes.data)
    assert rc in (0, 2), lib.emu_message().decode()
    return (scores, plan) if rc == 0 else None


@pytest.mark.parametrize("flags", [0, 1])
@pytest.mark.parametrize("depth,trees,features,values", [
    (3, 1, 1, None), (3, 15, 5, VALUES), (3, 16, 144, None), (3, 17, 145, VALUES), (3, 40, 288, VALUES),
    (3, 40, 289, None), (3, 600, 7, VALUES), (2, 31, 3, VALUES), (2, 33, 144, None), (2, 65, 576, VALUES),
])
def test_uniform_tables(emu, depth, trees, features, values, flags):
    ens = W.random_ensemble(depth * 100 + trees, trees, features, 1, 1 << depth, depth, values)
    deepest = W.random_ensemble(7, 1, features, 1 << depth, 1 << depth, depth, values)  # a complete one
    ens = W.Ensemble(np.concatenate([deepest.tree_offsets[:-1], ens.tree_offsets + deepest.n_nodes]),
                     *[np.concatenate([getattr(deepest, k), getattr(ens, k)])
                       for k in ("feature", "threshold", "left", "right", "value")], features)
    ens.feature[0] = features - 1  # the widest column is read
    X = W.random_docs(trees, 40, features, None if values is None else np.append(values, np.float32(np.nan)))
    got = _uniform(emu, ens, X, flags)
    assert got is not None
    scores, plan = got
    assert plan[0] == depth and plan[1] == (512 if features <= 144 else 256 if features <= 288 else 128)
    ref, _, _ = oracle.score(ens, X, rule=flags)
    np.testing.assert_allclose(scores, ref, rtol=1e-12, atol=1e-12)


def test_models_without_uniform_tables(emu):
    X = np.zeros((1, 600), np.float32)
    deep = W.random_ensemble(1, 20, 30, 16, 16, 4)
    stumps = W.random_ensemble(2, 20, 30, 2, 2)
    wide = W.random_ensemble(3, 20, 600, 8, 8, 3)
    wide.feature[0] = 576  # one column past the narrowest tile
    many = W.random_ensemble(4, 300, 1, 8, 8, 3)  # 2,100 distinct thresholds on one feature
    for ens in (deep, stumps, wide, many):
        assert _uniform(emu, ens, X[:, :ens.n_features].copy(), 0) is None
