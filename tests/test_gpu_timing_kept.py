"""Kernel timing on a table with kept rows and the bound off: both of the launch's passes are in it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1210_5128_amd import datagen

pytestmark = pytest.mark.gpu


def test_both_passes_are_timed():
    # 26 nodes, 15,276 entries per row, 64 copies of each of 512 orders: the whole call's time, by events around
    # many calls, is the two passes', the merge's and their gaps'; the streaming pass alone is well under it
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5128_amd import bnos
    n, B, reps = 26, 32768, 8
    net = datagen.random_network(n, 200, (2, 3), 3, seed=4)
    t = bnos.build_score_table(net.data, net.arities, 4)
    try:
        assert t.kept_entries() > 1000 * n
        t.score_bound(False)
        t.set_launch(B, chunk_steps=t_chunk(t))
        orders = torch.from_numpy(np.repeat(datagen.random_orders(n, 512, seed=2), B // 512, axis=0)).cuda()
        lse = torch.empty(B, dtype=torch.float64, device="cuda")
        mx, best = torch.empty_like(lse), torch.empty((B, n), dtype=torch.int64, device="cuda")
        t.score_orders(orders, lse, mx, best)
        torch.cuda.synchronize()
        t.timing(True)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(reps):
            t.score_orders(orders, lse, mx, best)
        e1.record()
        torch.cuda.synchronize()
        total = e0.elapsed_time(e1) / reps
        ms, launches, _ = t.timing_read()
        t.timing(False)
        print("total", total, "timed", ms / launches)
        assert launches == reps
        assert 0.85 * total < ms / launches <= total
    finally:
        t.free()


def t_chunk(t):
    """The longest chunk a launch of this table takes: few partials for the merge."""
    c = 16
    while c > 1:
        try:
            t.set_launch(1, chunk_steps=c)
            t.set_launch(1)
            return c
        except Exception:
            c //= 2
    return 1
