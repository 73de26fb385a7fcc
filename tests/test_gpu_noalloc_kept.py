"""Scoring without allocation on a table with kept rows, the score bound off: bit for bit what the allocating
call gives, up to the most orders it takes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1210_5128_amd import datagen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,K", [(20, 4), (33, 2), (64, 2)])
def test_most_orders_without_allocation(n, K):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5128_amd import bnos
    net = datagen.random_network(n, 500, (2, 3), 3, seed=n)
    t = bnos.build_score_table(net.data, net.arities, K)
    try:
        assert t.kept_entries() > 0
        t.score_bound(False)

        def score(call, B):
            out = [torch.full((B,), -1.0, dtype=torch.float64, device="cuda") for _ in range(2)]
            out += [torch.zeros((B, n), dtype=torch.int64, device="cuda"),
                    torch.zeros((B, n), dtype=torch.float64, device="cuda"),
                    torch.zeros((B, n), dtype=torch.float32, device="cuda")]
            call(orders[:B], *out)
            return out

        g = torch.Generator(device="cuda").manual_seed(2)
        orders = torch.rand((1 << 16, n), device="cuda", generator=g).argsort(dim=1).to(torch.int32)
        lo, hi = 1, 1 << 16                   # the most orders accepted
        while hi - lo > 1:
            mid = (lo + hi) // 2
            try:
                score(t.score_orders_noalloc, mid)
                lo = mid
            except bnos.BnosError as e:
                assert e.status == bnos.E_RANGE
                hi = mid
        for B in (lo, lo - 1, lo // 2 + 1, 16):
            for a, b in zip(score(t.score_orders_noalloc, B), score(t.score_orders, B)):
                assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), B
    finally:
        t.free()
