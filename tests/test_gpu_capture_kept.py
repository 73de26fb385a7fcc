"""A captured scoring launch on kept rows outlives calls on the same table that need a larger workspace."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1210_5128_amd import datagen

pytestmark = pytest.mark.gpu


def test_captured_scoring_after_streamed_calls():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5128_amd import bnos
    n, B = 33, 8
    net = datagen.random_network(n, 300, (2, 3), 3, seed=5)
    t = bnos.build_score_table(net.data, net.arities, 3)
    assert t.kept_entries() // 256 > 128                 # with partials: not one block per order
    orders = torch.from_numpy(datagen.random_orders(n, 5 * B, seed=1)).cuda().view(5, B, n)
    now = orders[0].clone()
    lse = torch.empty(B, dtype=torch.float64, device="cuda")
    mx, best = torch.empty_like(lse), torch.empty((B, n), dtype=torch.int64, device="cuda")
    want = []
    for k in range(5):                                   # also the warm-up that sizes the workspace
        t.score_orders(orders[k].contiguous(), lse, mx, best)
        want.append((lse.clone(), mx.clone(), best.clone()))
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        t.score_orders(now, lse, mx, best, stream=torch.cuda.current_stream())
    for k in range(5):
        if k == 1:
            t.score_bound(False)                         # the streaming pass's partials
            t.score_orders(orders[k].contiguous(), *[x.clone() for x in want[k]])
            t.score_bound(True)
        elif k == 2:
            t.autotune(orders[k].contiguous(), reps=2)
        elif k == 3:
            st = t.new_chain_state(48, 20)
            t.score_bound(False)
            t.run_chains(st, 20, 3)
            t.score_bound(True)
        now.copy_(orders[k])
        for x in (lse, mx, best):
            x.zero_()
        g.replay()
        torch.cuda.synchronize()
        for got, w in zip((lse, mx, best), want[k]):
            assert torch.equal(got, w), k
    del g
    t.free()
