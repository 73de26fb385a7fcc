"""Calls whose (order or chain, node) pairs are more than one launch can hold as a wavefront each (2^32
work-items): they run, and give what smaller calls give."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1210_5128_amd import datagen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bnos():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5128_amd import bnos as b
    return b


def test_many_chains_on_kept_rows_with_the_bound_off(bnos):
    # 57 tables x 65,536 chains x 18 nodes: 67,239,936 pairs, 4.3e9 work-items; the first, a middle and the
    # last table against the same chains on that table alone
    n, C, T, seed = 18, 65536, 57, 3
    tabs, states = [], []
    try:
        for k in range(T):
            net = datagen.random_network(n, 60, (2, 3), 3, seed=k)
            t = bnos.build_score_table(net.data, net.arities, 1)
            tabs.append(t)
            assert t.kept_entries() > 0
            t.score_bound(False)
            states.append(t.new_chain_state(C, 1))
        bnos.run_chains_multi(tabs, states, 1, seed)
        for k in (0, T // 2, T - 1):
            ref = tabs[k].new_chain_state(C, 1)
            tabs[k].run_chains(ref, 1, seed, chain_offset=k * C)
            torch.cuda.synchronize()
            for key in ("orders", "scores", "best_graphs", "best_scores", "accepted", "trace"):
                assert torch.equal(states[k][key], ref[key]), (k, key)
    finally:
        for t in tabs:
            t.free()


def test_most_orders_on_64_nodes(bnos):
    # 2^20 orders of 64 nodes: 2^26 pairs, 2^32 work-items; against the same orders in calls of 2^17
    n, B, step = 64, 1 << 20, 1 << 17
    net = datagen.random_network(n, 129, (2,), 3, seed=84)
    t = bnos.build_score_table(net.data, net.arities, 2)
    try:
        assert t.kept_entries() // 256 > 128             # more than one block per order scans
        g = torch.Generator(device="cuda").manual_seed(1)
        orders = torch.cat([torch.rand((step, n), device="cuda", generator=g).argsort(dim=1).to(torch.int32)
                            for _ in range(B // step)])

        def score(o):
            lse = torch.empty(o.shape[0], dtype=torch.float64, device="cuda")
            mx, best = torch.empty_like(lse), torch.empty(o.shape, dtype=torch.int64, device="cuda")
            t.score_orders(o, lse, mx, best)
            return lse, mx, best

        whole = score(orders)
        for b in range(0, B, step):
            part = score(orders[b:b + step])
            for w, p in zip(whole, part):
                assert torch.equal(w[b:b + step], p), b
        read, _ = t.count_tiles(orders)
        assert read == sum(t.count_tiles(orders[b:b + step])[0] for b in range(0, B, step))
    finally:
        t.free()


def test_more_chains_than_a_launch_holds_is_an_error(bnos):
    # 65 tables x 65,536 chains, a block of 1,024 threads each in the streamed sweep: 4.4e9 work-items, of
    # which a launch runs what is left modulo 2^32; the call is refused before any kernel runs
    n, C, T = 8, 65536, 65
    tabs, states = [], []
    try:
        for k in range(T):
            net = datagen.random_network(n, 40, (2,), 3, seed=k)
            t = bnos.build_score_table(net.data, net.arities, 1)
            tabs.append(t)
            t.score_bound(False)
            states.append(t.new_chain_state(C, 1))
        with pytest.raises(bnos.BnosError) as e:
            bnos.run_chains_multi(tabs, states, 1, 3)
        assert e.value.status == bnos.E_RANGE
        ref = tabs[0].new_chain_state(C, 1)               # and the next call is not disturbed
        tabs[0].run_chains(ref, 1, 3)
        assert torch.all(torch.isfinite(ref["scores"]))
    finally:
        for t in tabs:
            t.free()


def test_most_orders_on_64_nodes_streamed(bnos, monkeypatch):
    # the same 2^26 pairs where the score bound's cuts are computed ahead of the streaming pass
    if torch.cuda.mem_get_info()[0] < 160 << 30:
        pytest.skip("the partials of 2^20 orders take 104 GB")
    n, B, step = 64, 1 << 20, 1 << 17
    net = datagen.random_network(n, 129, (2,), 3, seed=84)
    t = bnos.build_score_table(net.data, net.arities, 2, chunk_steps=2)
    held = t.info()["device_bytes"]
    t.free()
    monkeypatch.setenv("BNOS_MAX_DEVICE_BYTES", str(held - 1))
    t = bnos.build_score_table(net.data, net.arities, 2, chunk_steps=2)
    monkeypatch.delenv("BNOS_MAX_DEVICE_BYTES")
    try:
        assert t.kept_entries() == 0
        g = torch.Generator(device="cuda").manual_seed(1)
        orders = torch.cat([torch.rand((step, n), device="cuda", generator=g).argsort(dim=1).to(torch.int32)
                            for _ in range(B // step)])

        def score(o):
            lse = torch.empty(o.shape[0], dtype=torch.float64, device="cuda")
            mx, best = torch.empty_like(lse), torch.empty(o.shape, dtype=torch.int64, device="cuda")
            t.score_orders(o, lse, mx, best)
            return lse, mx, best

        parts = [score(orders[b:b + step]) for b in range(0, B, step)]
        whole = score(orders)
        for k, b in enumerate(range(0, B, step)):
            for w, p in zip(whole, parts[k]):
                assert torch.equal(w[b:b + step], p), b
    finally:
        t.free()
