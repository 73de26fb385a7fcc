"""Scoring and chains from the kept rows (the entries no subset of theirs rules out), at the sizes
where their scan can go wrong: rows of one step, of many, of several sort runs, and rows too long
to be kept; every number of wavefronts per row."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1210_5128_amd import datagen

from test_gpu_parity import check_orders_against_oracle, dev_score, same_bits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bnos():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5128_amd import bnos as b
    return b


# (n, K, N, arities): a row of one entry; 64, 512 and 513 entries; one row per wavefront and more; kept
# rows of several thousand entries; rows too long to be kept (26, 22 and 48 nodes); 7,343 of 396,607 entries
# with single rows of several sort runs; no data, where every score ties
SHAPES = [(1, 0, 20, (2,)), (7, 6, 100, (2,)), (10, 6, 60, (2,)), (12, 4, 200, (2, 3)), (20, 4, 1000, (2,)),
          (33, 3, 80, (2,)), (26, 5, 300, (2,)), (36, 4, 2000, (2, 3, 4)), (22, 4, 300, (2,)),
          (57, 4, 1066, (2, 3, 4)), (64, 2, 129, (2,)), (48, 4, 60, (2,)), (9, 4, 0, (2, 3))]


@pytest.mark.parametrize("n,K,N,arities", SHAPES)
def test_kept_rows_against_streaming_and_oracle(bnos, n, K, N, arities):
    # with the bound off the streaming pass adds every entry that was not kept: bitwise equal, whatever
    # the number of orders (8, 4, 2 or 1 wavefronts per row, or one block per order); and the oracle
    net = datagen.random_network(n, N, arities, min(3, n - 1), seed=n + 10 * K)
    t = bnos.build_score_table(net.data, net.arities, K)
    orc = oracle.build_table(net.data, net.arities, K) if n <= 20 else None
    try:
        for B in (1, 6, 70, 700):
            orders = datagen.random_orders(n, B, seed=n + B)
            got = dev_score(t, orders)
            t.score_bound(False)
            plain = dev_score(t, orders)
            t.score_bound(True)
            same_bits(got, plain)
            if orc is not None and B == 6:
                assert check_orders_against_oracle(got, orc, K, orders) == 0
            if t.kept_entries():          # an order's result does not depend on the batch it is in
                one = dev_score(t, orders[B // 2:B // 2 + 1])
                same_bits(one, {k: v[B // 2:B // 2 + 1] for k, v in got.items()})
    finally:
        t.free()


def test_kept_rows_invalid_orders_and_memory_cap(bnos, monkeypatch):
    # an order that is not a permutation gives NaN and leaves the others alone; a table built under a
    # memory cap that has no room for kept rows scores the same (to the association of FP32 sums)
    net = datagen.random_network(24, 1500, (2, 3, 4), 3, seed=8)
    t = bnos.build_score_table(net.data, net.arities, 4)
    orders = datagen.random_orders(24, 9, seed=2)
    bad = orders.copy()
    bad[3, 0], bad[5, 7], bad[7, 2] = bad[3, 1], -1, 24
    got, ref = dev_score(t, bad), dev_score(t, orders)
    for b in range(9):
        if b in (3, 5, 7):
            assert np.isnan(got["lse"][b]) and np.isnan(got["max"][b]) and np.all(got["best"][b] == 0)
        else:
            same_bits({k: v[b:b + 1] for k, v in got.items()}, {k: v[b:b + 1] for k, v in ref.items()})
    held = t.info()["device_bytes"]
    assert t.kept_entries() > 0
    monkeypatch.setenv("BNOS_MAX_DEVICE_BYTES", str(held - 100000))
    c = bnos.build_score_table(net.data, net.arities, 4)
    assert c.kept_entries() == 0 and c.info()["device_bytes"] <= held - 100000
    out = dev_score(c, orders)
    assert np.array_equal(out["best"], ref["best"])
    assert np.array_equal(out["node_second"].view(np.uint32), ref["node_second"].view(np.uint32))
    np.testing.assert_allclose(out["node_lse"], ref["node_lse"], rtol=0, atol=2e-6)
    t.free()
    c.free()


@pytest.mark.parametrize("n,K,N,arities,chains", [(2, 1, 50, (2,), 3), (9, 4, 0, (2, 3), 5), (20, 4, 1000, (2,), 4),
                                                  (24, 4, 1500, (2, 3, 4), 600), (64, 2, 129, (2,), 7)])
@pytest.mark.parametrize("target", [0, 1])
def test_kept_chains_take_the_streamed_decisions(bnos, n, K, N, arities, chains, target):
    # the one-launch chains against the launch-per-iteration sweep (score bound off): the same moves and, bit
    # for bit, the same traces, records and traced edges, whole and resumed at an odd place
    net = datagen.random_network(n, N, arities, min(3, n - 1), seed=3 * n + K)
    t = bnos.build_score_table(net.data, net.arities, K)
    assert t.kept_entries() > 0
    iters, cut, every = 150, 67, 1
    edges = [(0, 1), (1, 0)]
    out = []
    try:
        for on in (True, False):
            t.score_bound(on)
            st = t.new_chain_state(chains, iters, flags=True, topk=3, edges=edges, harvest_cap=20)
            t.run_chains(st, iters, seed=77, target=target, chain_offset=5)
            torch.cuda.synchronize()
            out.append({k: v.cpu().numpy() for k, v in st.items() if torch.is_tensor(v)})
        a, b = out
        for k in a:
            assert np.array_equal(a[k].view(np.uint8), b[k].view(np.uint8)), k
        t.score_bound(True)
        st = t.new_chain_state(chains, cut, flags=True, topk=3)
        t.run_chains(st, cut, seed=77, target=target, chain_offset=5)
        st2 = t.new_chain_state(chains, iters - cut, flags=True, topk=3)
        for k in ("orders", "scores", "best_graphs", "best_scores", "accepted", "top_graphs", "top_scores", "top_count"):
            st2[k] = st[k]
        t.run_chains(st2, iters - cut, seed=77, target=target, chain_offset=5, first_iteration=cut)
        torch.cuda.synchronize()
        for k in ("orders", "scores", "best_graphs", "best_scores", "accepted", "top_graphs", "top_scores", "top_count"):
            assert np.array_equal(st2[k].cpu().numpy(), a[k]), k
        assert np.array_equal(st2["accept_flags"].cpu().numpy(), a["accept_flags"][:, cut:])
        assert np.array_equal(st2["trace"].cpu().numpy(), a["trace"][:, cut:])
    finally:
        t.free()


def test_kept_and_streamed_tables_in_one_call(bnos):
    # tables with and without kept rows, and one with the bound off, advanced together: each as by itself
    shapes = [(12, 3, 300, (2, 3)), (48, 4, 60, (2,)), (20, 4, 1000, (3,))]
    tabs = []
    for n, K, N, ar in shapes:
        net = datagen.random_network(n, N, ar, 3, seed=n)
        tabs.append(bnos.build_score_table(net.data, net.arities, K))
    assert [t.kept_entries() > 0 for t in tabs] == [True, False, True]
    tabs[2].score_bound(False)
    states = [t.new_chain_state(5, 40, flags=True) for t in tabs]
    bnos.run_chains_multi(tabs, states, 40, 9, chain_offset=2)
    torch.cuda.synchronize()
    for k, t in enumerate(tabs):
        ref = t.new_chain_state(5, 40, flags=True)
        t.run_chains(ref, 40, 9, chain_offset=2 + 5 * k)
        torch.cuda.synchronize()
        for key in ("orders", "scores", "best_graphs", "best_scores", "accepted", "trace", "accept_flags"):
            assert torch.equal(states[k][key], ref[key]), (k, key)
    for t in tabs:
        t.free()


@pytest.mark.parametrize("chains", [1, 3, 4])
def test_few_chains_on_long_kept_rows(bnos, chains):
    # below 4 chains such a table is streamed: the same moves as on its kept rows (the sums differ in
    # FP32 association, so a decision could differ where ln u is within about 1e-4 of the difference: not
    # at this seed's few iterations), and a resumed run continues the whole one bit for bit
    net = datagen.random_network(57, 1066, (2, 3, 4), 3, seed=68)
    t = bnos.build_score_table(net.data, net.arities, 4)
    try:
        assert t.kept_entries() // 256 > 1600
        whole = t.new_chain_state(chains, 40)
        t.run_chains(whole, 40, 5)
        parts = t.new_chain_state(chains, 40)
        t.run_chains(parts, 23, 5)
        t.run_chains(parts, 17, 5, first_iteration=23)
        many = t.new_chain_state(4, 40)
        t.run_chains(many, 40, 5)
        for k in ("orders", "scores", "best_scores", "best_graphs", "accepted"):
            assert torch.equal(whole[k], parts[k]), k
        assert torch.equal(whole["orders"], many["orders"][:chains])
        assert torch.allclose(whole["scores"], many["scores"][:chains], rtol=1e-6)
        assert torch.equal(whole["best_graphs"], many["best_graphs"][:chains])
    finally:
        t.free()
