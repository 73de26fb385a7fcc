"""Scoring one order from host arrays: the same numbers, bit for bit, as the call on device tensors,
for the smallest and the largest node counts and from several threads on one table."""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1210_5128_amd import datagen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,K,N", [(2, 1, 50), (8, 3, 200), (33, 3, 300), (64, 2, 200)])
def test_host_order_equals_device_order(n, K, N):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5128_amd import bnos
    rng = np.random.default_rng(n)
    data = rng.integers(0, 2, size=(N, n)).astype(np.int8)
    t = bnos.build_score_table(data, np.full(n, 2, np.int32), K)
    B = 12
    orders = np.ascontiguousarray(datagen.random_orders(n, B, n + 1), dtype=np.int32)
    d = torch.from_numpy(orders).cuda()
    want = []
    for b in range(B):                              # one order per call: the same launch shape
        lse, mx = (torch.empty(1, dtype=torch.float64, device="cuda") for _ in range(2))
        best = torch.empty((1, n), dtype=torch.int64, device="cuda")
        t.score_orders(d[b:b + 1].contiguous(), lse, mx, best)
        want.append((lse.item(), mx.item(), best.cpu().numpy().view(np.uint64)[0]))
    got = [None] * B

    def work(k):
        for b in range(k, B, 4):
            got[b] = t.score_order(orders[b])

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    for g, w in zip(got, want):
        assert g[0] == w[0] and g[1] == w[1]
        assert np.array_equal(g[2], w[2])
    with pytest.raises(Exception):
        t.score_order(np.zeros(n, np.int32))        # not a permutation
    t.free()
