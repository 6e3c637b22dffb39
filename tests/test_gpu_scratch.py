"""Device memory that calls borrow (positions of leaf ids, rows of leaf vectors, threshold codes, split
sums): the calls return while earlier work of the stream still runs, keep their memory over a
synchronisation, give it back with the last handle, and don't share it between streams."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as W
from _gpu import assert_leaves_equal, assert_scores_close, dev

pytestmark = pytest.mark.gpu

# what the call is, trees, features, leaves, depth, documents, outputs
CALLS = [
    ("leaf positions", 300, 20, 8, None, 20_000, 1),
    ("leaf rows", 200, 20, 8, None, 30_000, 6),
    ("shallow codes", 2_000, 30, 8, 3, 60_000, 1),
    ("terminal codes", 64, 500, 250, None, 40_000, 1),
]


@pytest.fixture(scope="module")
def T():
    import paper_1212_2287_amd as T
    T.load_library()
    return T


def _model(T, trees, features, leaves, depth, n_out):
    ens = W.random_ensemble(trees + n_out, trees, features, leaves, leaves, depth)
    vals = W.make_leaf_vectors(ens, n_out, "dense", seed=1) if n_out > 1 else None
    return ens, vals, (T.TreeEnsemble.from_ensemble(ens, leaf_values=vals) if n_out > 1 else T.TreeEnsemble.from_ensemble(ens))


def _call(m, what):
    return m.predict_leaves if what == "leaf positions" else m.predict


@pytest.mark.parametrize("what,trees,features,leaves,depth,docs,n_out", CALLS, ids=[c[0] for c in CALLS])
def test_calls_return_without_waiting(T, what, trees, features, leaves, depth, docs, n_out):
    import torch
    _, _, m = _model(T, trees, features, leaves, depth, n_out)
    a = torch.randn(8192, 8192, device="cuda")
    c = torch.empty_like(a)
    with m:
        x = torch.rand((docs, features), device="cuda")
        out = _call(m, what)(x)  # the first call may allocate
        torch.mm(a, a, out=c)
        torch.cuda.synchronize()
        for _ in range(20):  # over 100 ms
            torch.mm(a, a, out=c)
        before = torch.cuda.Event()
        before.record()
        _call(m, what)(x, out)
        _call(m, what)(x, out)
        assert not before.query(), "the call waited for the stream"
        torch.cuda.synchronize()


@pytest.mark.parametrize("what,trees,features,leaves,depth,docs,n_out", CALLS, ids=[c[0] for c in CALLS])
def test_memory_is_kept_between_calls_and_given_back(T, what, trees, features, leaves, depth, docs, n_out):
    import torch
    _, _, m = _model(T, trees, features, leaves, depth, n_out)
    with m:
        x = torch.rand((docs, features), device="cuda")
        out = _call(m, what)(x)
        torch.cuda.synchronize()
        idle = torch.cuda.mem_get_info()[0]
        small = _call(m, what)(x[:docs // 2].contiguous())
        kept = []
        for _ in range(4):
            _call(m, what)(x, out)
            torch.cuda.synchronize()
            kept.append(torch.cuda.mem_get_info()[0])
        del small
        assert len(set(kept)) == 1
    del m
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] >= idle + (2 << 20), "the handle's memory and the calls'"


@pytest.mark.parametrize("what,trees,features,leaves,depth,docs,n_out", CALLS, ids=[c[0] for c in CALLS])
def test_streams_do_not_share_memory(T, what, trees, features, leaves, depth, docs, n_out):
    """Three streams with batches of their own, the handle's calls in turn without a synchronisation."""
    import torch
    ens, vals, m = _model(T, trees, features, leaves, depth, n_out)
    sizes = [docs, docs - 77, docs // 2 + 5]
    X = [W.random_docs(n, n, features) for n in sizes]
    with m:
        x = [dev(v) for v in X]
        streams = [torch.cuda.Stream() for _ in sizes]
        outs = [[] for _ in sizes]
        torch.cuda.synchronize()
        for _ in range(6):
            for s, v, o in zip(streams, x, outs):
                with torch.cuda.stream(s):
                    o.append(_call(m, what)(v))
        torch.cuda.synchronize()
        for v, o in zip(X, outs):
            assert all(torch.equal(r, o[0]) for r in o)
            got = o[0].cpu().numpy()
            if what == "leaf positions":
                assert_leaves_equal(got, oracle.score(ens, v)[1], what)
            elif n_out > 1:
                ref = oracle.score_multi(ens, vals, v)
                for c in range(n_out):
                    assert_scores_close(got[:, c], ref[:, c], what)
            else:
                assert_scores_close(got, oracle.score(ens, v)[0], what)


def _fill_up_to(left, what):
    """Tensors that leave `left` bytes of the device's memory free (8 MiB more or less)."""
    import torch
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    fill, slack = [], 8 << 20
    for _ in range(4):  # the first figure can lag behind memory given back
        free = torch.cuda.mem_get_info()[0]
        if free > left + slack:
            fill.append(torch.empty(free - left, dtype=torch.uint8, device="cuda"))
    print(f"[scratch] {what}, {free >> 20} MiB free", flush=True)
    assert left - slack <= free <= left + slack
    return fill


@pytest.mark.parametrize("n_out", [1, 6])
def test_room_for_the_codes_alone_is_enough(T, n_out):
    """A coded model on a device with room for its codes, but not for positions and codes: the walk
    stores its results directly, as it does for small batches."""
    import torch
    ens = W.random_ensemble(11, 200, 500, 250, 250)
    docs, mib = 100_000, 1 << 20  # 38 MiB of positions, 95 MiB of codes
    vals = W.make_leaf_vectors(ens, n_out, "dense", seed=1) if n_out > 1 else None

    def handle():
        return T.TreeEnsemble.from_ensemble(ens, leaf_values=vals) if n_out > 1 else T.TreeEnsemble.from_ensemble(ens)
    x = torch.rand((docs, 500), device="cuda")
    small = x[:21_000].contiguous()
    with handle() as m:
        ref = (m.predict if n_out > 1 else m.predict_leaves)(x)
        torch.cuda.synchronize()
    with handle() as m:
        call = m.predict if n_out > 1 else m.predict_leaves
        out = torch.zeros_like(ref)
        few = call(small)  # kernels loaded, 29 MiB in the pool
        call(small[:500].contiguous())
        fill = _fill_up_to(80 * mib, f"{n_out} outputs")
        call(x, out)
        torch.cuda.synchronize()
        del fill, few
        torch.cuda.empty_cache()
        if n_out == 1:
            assert torch.equal(out, ref)
        else:
            assert torch.allclose(out, ref, rtol=1e-5, atol=1e-6)
        call(x, out)  # and with room again
        torch.cuda.synchronize()
        assert torch.equal(out, ref)


def test_each_threads_own_default_stream(T):
    """hipStreamPerThread is one value for a stream of each thread: split batches of one handle from four
    threads share the handle's scratch one after another."""
    import threading

    import torch
    per_thread = 2  # hipStreamPerThread
    ens = W.random_ensemble(21, 1_000, 136, 32, 32)
    n = 60
    with T.TreeEnsemble.from_ensemble(ens) as m:
        xs = [dev(W.random_docs(100 + i, n, 136)) for i in range(4)]
        refs = [m.predict(x).clone() for x in xs]
        outs = [torch.zeros((40, n), device="cuda") for _ in xs]
        torch.cuda.synchronize()
        errors = []

        def work(i):
            try:
                for o in outs[i]:
                    m.predict(xs[i], o, stream=per_thread)
            except Exception as e:  # noqa: BLE001
                errors.append(e)
        threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
        for t in threads:
            t.start()
        for t in threads:
            t.join(60)
        assert not errors and not any(t.is_alive() for t in threads)
        torch.cuda.synchronize()
        for o, r in zip(outs, refs):
            assert all(torch.equal(row, r) for row in o)


def test_eager_calls_during_a_capture(T):
    """A call on another stream that makes the pool grow while a graph is being captured: it runs at once and
    leaves the capture whole."""
    import torch
    ens = W.random_ensemble(31, 300, 20, 8, 8)
    x, big = torch.rand((20_000, 20), device="cuda"), torch.rand((30_000, 20), device="cuda")
    with T.TreeEnsemble.from_ensemble(ens) as m:
        ref, ids_ref = m.predict(x), m.predict_leaves(big)
        torch.cuda.synchronize()
    with T.TreeEnsemble.from_ensemble(ens) as m:  # a new pool
        m.predict(x[:100].contiguous())
        out, ids, other = torch.zeros_like(ref), torch.zeros_like(ids_ref), torch.cuda.Stream()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            m.predict(x, out)
            m.predict_leaves(big, ids, stream=other)
            m.predict(x, out)
        for _ in range(2):
            out.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, ref)
        assert torch.equal(ids, ids_ref)


@pytest.mark.parametrize("what", ["larger than the pool keeps", "captured", "a new model"])
def test_memory_the_pool_holds_is_there_for_others(T, what):
    """256 MiB idle in the pool and 400 MiB free: allocations of about 550 MiB outside the pool get both."""
    import torch
    mib = 1 << 20
    ids = W.random_ensemble(41, 2_000, 30, 3, 3)
    coded = W.random_ensemble(42, 64, 500, 250, 250)
    docs = 575_000  # 548 MiB of codes
    x = torch.rand((docs, 500), device="cuda")
    out = torch.zeros(docs, device="cuda")
    if what == "a new model":  # 960,000 leaf rows of 116 floats, 425 MiB, and its records
        base, n = W.random_ensemble(43, 100, 20, 64, 64), 15_000
        each = [base.tree(t % 100) for t in range(n)]
        wide = W.Ensemble(np.arange(n + 1, dtype=np.int64) * 127,
                          *[np.concatenate([t[k] for t in each]) for k in range(5)], 20)
        vals = np.zeros((wide.n_nodes, 116), np.float32)
        vals[:, 3] = wide.value
    with T.TreeEnsemble.from_ensemble(ids) as m, T.TreeEnsemble.from_ensemble(coded) as c:
        ref = c.predict(x).clone()
        big = torch.rand((70_000, 30), device="cuda")
        got = m.predict_leaves(big)  # 256 MiB of positions
        assert m.last_path() == T.TREE_ENS_PATH_ROWS
        torch.cuda.synchronize()
        del got
        fill = _fill_up_to(400 * mib, what)
        if what == "larger than the pool keeps":
            c.predict(x, out)
        elif what == "captured":
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                c.predict(x, out)
            g.replay()
        else:
            w = T.TreeEnsemble.from_ensemble(wide, leaf_values=vals)
            del fill
            few = big[:100, :20].contiguous()
            scores = w.predict(few)
            torch.cuda.synchronize()
            assert_scores_close(scores[:, 3].cpu().numpy(), oracle.score(wide, few.cpu().numpy())[0], what)
            w.close()
            return
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
        del fill
        torch.cuda.empty_cache()
