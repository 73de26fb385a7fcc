"""The launch-per-iteration sweep and the streaming pass with the score bound on, on tables that list no kept
rows (a memory cap just below their size), and chains on kept rows over several launches."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1210_5128_amd import datagen

from test_gpu_chains import compare_chains, gpu_chains
from test_gpu_kept import SHAPES
from test_gpu_learned import dyadic_position_network, oracle_learned_step
from test_gpu_parity import check_orders_against_oracle, dev_score, same_bits

pytestmark = pytest.mark.gpu

REL = 1e-5


@pytest.fixture(scope="module")
def bnos():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5128_amd import bnos as b
    return b


def streamed(bnos, monkeypatch, w, **opts):
    """The workload's table without kept rows: built under a cap one byte below the table with them."""
    net, prior = datagen.make(w)
    t = bnos.build_score_table(net.data, net.arities, w.K, prior=prior, **opts)
    assert t.kept_entries() > 0
    held = t.info()["device_bytes"]
    t.free()
    monkeypatch.setenv("BNOS_MAX_DEVICE_BYTES", str(held - 1))
    t = bnos.build_score_table(net.data, net.arities, w.K, prior=prior, **opts)
    monkeypatch.delenv("BNOS_MAX_DEVICE_BYTES")
    assert t.kept_entries() == 0
    return t


@pytest.fixture(scope="module")
def oracles():
    out = {}
    for name in ("tiny8", "prior20"):
        w = datagen.WORKLOADS[name]
        net, prior = datagen.make(w)
        out[name] = oracle.build_table(net.data, net.arities, w.K, prior=prior)
    return out


@pytest.mark.parametrize("chunk_steps", [1, 2, 4, 16])
def test_scoring_shapes(bnos, oracles, monkeypatch, chunk_steps):
    # every chunk length and number of orders per block: the oracle's result, bound on and off the same bits
    w = datagen.WORKLOADS["prior20"]
    t = streamed(bnos, monkeypatch, w, chunk_steps=chunk_steps)
    try:
        orders = datagen.random_orders(w.n, 11, seed=60 + chunk_steps)
        for bt in (1, 2, 4, 8):
            t.set_launch(11, orders_per_block=bt)
            on = dev_score(t, orders)
            assert check_orders_against_oracle(on, oracles["prior20"], w.K, orders) == 0
            t.score_bound(False)
            same_bits(on, dev_score(t, orders))
            t.score_bound(True)
    finally:
        t.free()


@pytest.mark.parametrize("bt", [1, 2, 4, 8])
def test_chain_shapes(bnos, oracles, monkeypatch, bt):
    # chains per scoring block and iterations per graph: the oracle's chains, and the same bits whatever the graphs
    w = datagen.WORKLOADS["tiny8"]
    t = streamed(bnos, monkeypatch, w)
    try:
        C, iters = 12, 601
        t.set_launch(C, orders_per_block=bt)
        ref = gpu_chains(t, C, iters, seed=203 + bt, topk=4)
        assert compare_chains(ref, oracles["tiny8"], w.K, 203 + bt, iters, 0, topk=4) >= C - 1
        for sweep in (1, 7, 1000):
            g = gpu_chains(t, C, iters, seed=203 + bt, sweep_len=sweep, topk=4)
            for k in g:
                if g[k] is not None and hasattr(g[k], "view"):
                    assert np.array_equal(g[k].view(np.uint8), ref[k].view(np.uint8)), (sweep, k)
        # resumed at an odd place
        st = t.new_chain_state(C, 120, flags=True)
        t.run_chains(st, 120, 203 + bt)
        st["trace"] = torch.zeros((C, 482), dtype=torch.float64, device="cuda")
        st["accept_flags"] = torch.zeros((C, 481), dtype=torch.uint8, device="cuda")
        t.run_chains(st, 481, 203 + bt, first_iteration=120)
        torch.cuda.synchronize()
        for k in ("orders", "scores", "best_graphs", "best_scores", "accepted"):
            assert np.array_equal(st[k].cpu().numpy(), ref[k]), k
        assert np.array_equal(st["trace"].cpu().numpy(), ref["trace"][:, 120:])
        assert np.array_equal(st["accept_flags"].cpu().numpy(), ref["accept_flags"][:, 120:])
    finally:
        t.free()


@pytest.mark.parametrize("bt", [1, 2, 4, 8])
def test_chains_with_the_bound_on_and_off(bnos, monkeypatch, bt):
    w = datagen.WORKLOADS["mixed40"]
    t = streamed(bnos, monkeypatch, w)
    try:
        C, iters, runs = 64, 100, []
        t.chains_set_launch(C, 0, bt)
        for on in (False, True):
            t.score_bound(on)
            runs.append(gpu_chains(t, C, iters, seed=31))
        a, b = runs
        for k in ("accept_flags", "orders", "best_graphs", "best_scores", "accepted", "scores", "trace"):
            assert np.array_equal(a[k].view(np.uint8), b[k].view(np.uint8)), k
    finally:
        t.free()


@pytest.mark.parametrize("target", [0, 1])
def test_learned_chains_in_lockstep(bnos, oracles, monkeypatch, target):
    # as on kept rows: the same proposals, and the same decisions but within 1e-3 of the threshold
    w = datagen.WORKLOADS["tiny8"]
    t, orc = streamed(bnos, monkeypatch, w), oracles["tiny8"]
    stats = oracle.table_stats(orc, w.K, round_f32=True)
    prm = dyadic_position_network(31 + target)
    m = bnos.Mlp()
    m.set_params(prm.astype(np.float32), np.zeros(8, np.float32), np.ones(8, np.float32))
    try:
        C, iters, seed, eps = 6, 250, 87 + target, 0.25
        st = t.new_chain_state(C, iters, flags=True)
        t.run_chains(st, iters, seed=seed, target=target, mlp=m, eps=eps)
        g = {k: (v.cpu().numpy() if v is not None else None) for k, v in st.items()}
        full = 0
        for c in range(C):
            res = oracle.run_chain_learned(orc, w.K, seed, c, iters, prm, np.zeros(8), np.ones(8), None, stats,
                                           eps=eps, target=target)
            mism = np.nonzero(g["accept_flags"][c, :iters].astype(bool) != res["acc"].astype(bool))[0]
            if len(mism):
                k = int(mism[0]) + 1
                lu, ratio = oracle_learned_step(orc, w.K, seed, c, k, res, prm, stats, eps, target)
                assert abs(lu - ratio) <= 1e-3, (c, k, lu, ratio)
                continue
            full += 1
            np.testing.assert_allclose(g["trace"][c, :iters + 1], res["trace"], rtol=REL, atol=1e-6)
            assert list(g["orders"][c]) == list(res["order"]), c
            assert [int(x) for x in g["best_graphs"][c].view(np.uint64)] == [int(x) for x in res["best_graph"]], c
        assert full >= C - 1
    finally:
        m.free()
        t.free()


@pytest.mark.parametrize("learned", [False, True])
def test_more_iterations_than_one_launch_on_kept_rows(bnos, learned):
    # 9,001 iterations are three launches of at most 4,096: the same as two calls that end elsewhere
    w = datagen.WORKLOADS["tiny8"]
    net, prior = datagen.make(w)
    t = bnos.build_score_table(net.data, net.arities, w.K, prior=prior)
    m = None
    if learned:
        m = bnos.Mlp()
        m.set_params(datagen.mlp_params(3, scale=0.3).astype(np.float32), np.zeros(8, np.float32),
                     np.array([1, 100, 100, 1, 1, 100, 100, 100], np.float32))
    try:
        assert t.kept_entries() > 0
        C, iters, cut, every, seed = 5, 9001, 5001, 3, 17
        edges = [(0, 1), (5, 2)]

        def run(state, k, first):
            t.run_chains(state, k, seed, first_iteration=first, trace_every=every, mlp=m)
            torch.cuda.synchronize()

        whole = t.new_chain_state(C, iters, trace_every=every, flags=True, topk=5, edges=edges, harvest_cap=40)
        run(whole, iters, 0)
        a = t.new_chain_state(C, cut, trace_every=every, flags=True, topk=5, edges=edges, harvest_cap=40)
        run(a, cut, 0)
        b = t.new_chain_state(C, iters - cut, trace_every=every, flags=True, topk=5, edges=edges, harvest_cap=40)
        own = ("trace", "accept_flags", "edge_trace")
        for k, v in a.items():
            if k not in own:
                b[k] = v
        run(b, iters - cut, cut)
        assert int(whole["accepted"].min()) > 0
        for k, v in whole.items():
            if torch.is_tensor(v) and k not in own:
                assert torch.equal(v, b[k]), k
        for k in ("trace", "edge_trace"):
            n = cut // every
            assert torch.equal(whole[k][:, :n + 1], a[k]), k
            assert torch.equal(whole[k][:, n + 1:], b[k][:, 1:]), k      # (entry 0 of a resumed call: its start)
        assert torch.equal(whole["accept_flags"], torch.cat([a["accept_flags"], b["accept_flags"]], dim=1))
    finally:
        if m is not None:
            m.free()
        t.free()


@pytest.mark.parametrize("n,K,N,arities", SHAPES)
def test_which_shapes_list_kept_rows(bnos, n, K, N, arities):
    # the tables that the tests of kept rows mean to be too long to be kept, and the others
    net = datagen.random_network(n, N, arities, min(3, n - 1), seed=n + 10 * K)
    t = bnos.build_score_table(net.data, net.arities, K)
    kept = t.kept_entries() > 0
    t.free()
    assert kept == ((n, K) not in ((26, 5), (22, 4), (48, 4)))
