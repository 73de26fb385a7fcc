"""The score bound leaves chains unchanged, bit for bit, whichever path serves them: on kept rows of more
than eight scan parts, and streamed whole where a table with kept rows has few chains."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1210_5128_amd import datagen

pytestmark = pytest.mark.gpu


# 1,665 and 753 steps of kept rows: streamed below 4 chains; 3,287 steps of rows of 425,924 entries
@pytest.mark.parametrize("n,K,N,seed,chains", [(57, 4, 1066, 68, 1), (57, 4, 1066, 68, 3), (57, 4, 1066, 68, 4),
                                               (57, 4, 1066, 68, 9), (45, 3, 290, 1, 3), (45, 3, 290, 1, 4),
                                               (58, 4, 587, 2, 15), (58, 4, 587, 2, 16)])
def test_bound_on_and_off_on_long_kept_rows(n, K, N, seed, chains):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5128_amd import bnos
    net = datagen.random_network(n, N, (2, 3, 4), 3, seed=seed)
    t = bnos.build_score_table(net.data, net.arities, K)
    try:
        assert t.kept_entries() > 0
        runs = []
        for on in (True, False):
            t.score_bound(on)
            st = t.new_chain_state(chains, 120, flags=True, topk=4)
            t.run_chains(st, 120, 21)
            torch.cuda.synchronize()
            runs.append({k: v.cpu().numpy() for k, v in st.items() if torch.is_tensor(v)})
        for k in runs[0]:
            assert np.array_equal(runs[0][k].view(np.uint8), runs[1][k].view(np.uint8)), k
    finally:
        t.free()
