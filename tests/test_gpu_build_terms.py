"""The table build's lookup terms as 64-bit integers and, where no integer unit serves, in FP64: every
entry against the oracle, and both counting modes bit for bit, at the edges of the integer rule (sample
size ess in [1e-6, 1e6]), of a wavefront's 64 cells and of a run of subsets."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1210_5128_amd import datagen

from test_gpu_parity import ulp32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bnos():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5128_amd import bnos as b
    return b


@pytest.mark.parametrize("n,K,N,arities,ess", [
    (9, 3, 700, (2, 5), 1.0), (9, 3, 700, (2, 5), 1e-6), (9, 3, 700, (2, 5), 9e-7), (9, 3, 700, (2, 5), 1e6),
    (9, 3, 700, (2, 5), 1.1e6), (8, 6, 1, (2,), 0.5), (9, 6, 300, (2, 3), 2.0), (7, 1, 257, (8,), 1.0),
    (6, 2, 255, (1, 4, 25), 1.0), (3, 2, 60, (25,), 3.0), (2, 1, 4000, (127,), 1.0), (1, 0, 5, (3,), 1.0),
    (22, 4, 64, (2,), 10.0)])
def test_entries_match_the_oracle(bnos, n, K, N, arities, ess):
    net = datagen.random_network(n, N, arities, min(3, n - 1), seed=n + N)
    prior = datagen.random_prior(n, seed=3)
    a = bnos.build_score_table(net.data, net.arities, K, ess=ess, prior=prior, log_gamma=-0.75)
    b = bnos.build_score_table(net.data, net.arities, K, ess=ess, prior=prior, log_gamma=-0.75, count_mode=1)
    orc = oracle.build_table(net.data, net.arities, K, ess=ess, prior=prior, log_gamma=-0.75)
    try:
        for i in range(n):
            masks, got = a.export(i)
            masks_b, other = b.export(i)
            assert np.array_equal(masks, masks_b) and np.array_equal(got.view(np.uint32), other.view(np.uint32)), i
            want = np.array([orc[i, oracle.rank(n, K, i, int(m))] for m in masks])
            # one FP32 rounding of a sum whose FP64 error stays far below half an ulp, and the oracle's own
            # lgamma differences: at large ess they lose ess ln(ess) 2^-52 per term
            slack = 2 * ulp32(want) + 1e-12 * max(1.0, ess) * max(1.0, abs(np.log(ess))) * min(N + 1, 16384)
            assert np.all(np.abs(got.astype(np.float64) - want) <= slack), (i, np.abs(got - want).max())
    finally:
        a.free()
        b.free()
