"""The autotuner on a table scored from its kept entries: the shape it leaves to the table's streamed calls
is one it has timed."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1210_5128_amd import datagen

from test_gpu_parity import dev_score, same_bits

pytestmark = pytest.mark.gpu


def test_streamed_shape_is_timed():
    # 30 nodes, 28 steps per row: two orders in 16-step chunks are 60 blocks and take half as long again as
    # in 1- to 8-step chunks (23 us against 15 to 18); the longest chunk was taken untimed
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5128_amd import bnos
    net = datagen.random_network(30, 1994, (2, 3, 4), 3, seed=30)
    t = bnos.build_score_table(net.data, net.arities, 4)
    try:
        assert t.kept_entries() > 0
        orders = datagen.random_orders(30, 2, seed=3)
        before = dev_score(t, orders)
        cs, bt, gather, ms = t.autotune(torch.from_numpy(orders).cuda(), reps=100)
        assert cs in (1, 2, 4, 8) and bt in (1, 2) and ms > 0
        if not gather:
            same_bits(dev_score(t, orders), before)
    finally:
        t.free()
