"""Terminal packets of coded models, walked on the host the way the kernel addresses them and compared
with the oracle: every shape of a terminal, trees on both sides of a window, cut trees, mixed sizes,
both tie rules and IEEE corner values."""
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
    lib.emu_term.argtypes = [ctypes.c_int32, P, P, P, P, P, P, ctypes.c_uint32, P, ctypes.c_int64, ctypes.c_int32, P, P]
    lib.emu_message.restype = ctypes.c_char_p
    return lib


def _term(lib, ens, X, flags):
    arrs = [np.ascontiguousarray(a, t) for a, t in ((ens.tree_offsets, np.int64), (ens.feature, np.int32),
            (ens.threshold, np.float32), (ens.left, np.int32), (ens.right, np.int32), (ens.value, np.float32))]
    scores, plan = np.empty(X.shape[0]), np.zeros(3, np.int32)
    rc = lib.emu_term(ens.n_trees, *[a.ctypes.data for a in arrs], flags, X.ctypes.data, X.shape[0], X.shape[1],
                      scores.ctypes.data, plan.ctypes.data)
    assert rc in (0, 2), lib.emu_message().decode()
    return (scores, plan) if rc == 0 else None


@pytest.mark.parametrize("trees,least,most,features,values,cut", [
    (70, 200, 256, 500, None, False), (65, 1, 512, 767, VALUES, True), (40, 250, 290, 700, VALUES, True),
    (300, 100, 260, 767, None, False), (33, 120, 700, 650, None, True), (20, 900, 1_300, 420, None, True),
])
@pytest.mark.parametrize("flags", [0, 1])
def test_term_packets(emu, trees, least, most, features, values, cut, flags):
    ens = W.random_ensemble(trees + most, trees, features, least, most, None, values)
    ens.feature[np.argmax(ens.feature >= 0)] = features - 1
    X = W.random_docs(trees, 30, features, None if values is None else np.append(values, np.float32(np.nan)))
    got = _term(emu, ens, X, flags)
    assert got is not None
    scores, plan = got
    assert plan[2] >= trees and (not cut or plan[2] > trees)
    ref, _, _ = oracle.score(ens, X, rule=flags)
    np.testing.assert_allclose(scores, ref, rtol=1e-12, atol=1e-12)


def test_models_without_term_packets(emu):
    X = np.zeros((1, 800), np.float32)
    narrow = W.random_ensemble(1, 40, 136, 256, 256)   # float documents
    wide = W.random_ensemble(2, 40, 800, 256, 256)     # the windows do not fit
    apart = W.random_ensemble(3, 40, 700, 4_000, 4_000)  # more than nine pieces per tree
    for ens in (narrow, wide, apart):
        assert _term(emu, ens, X[:, :ens.n_features].copy(), 0) is None
