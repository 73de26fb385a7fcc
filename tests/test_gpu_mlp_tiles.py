"""The network's kernels at the edges of their tiles: node counts about a 16-row tile, more samples
than one launch has blocks, and gradient blocks that are not full.  The forward pass is held
against itself (a sample's logits do not depend on the batch, bit for bit) and the FP64 oracle,
a training step against Adam applied to the gradient call's result."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1210_5128_amd import datagen
from test_gpu_mlp import bnos, oracle_params, rel, sample_inputs, N_PARAM  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,R", [(2, 3), (15, 1), (16, 2), (17, 515), (33, 9), (48, 17), (49, 8), (63, 513)])
def test_tiles(bnos, n, R):  # noqa: F811
    feats, pairs = sample_inputs(R, n, 100 + n)
    p32 = datagen.mlp_params(11).astype(np.float32)
    mu, sd = feats.reshape(-1, 8).mean(axis=0), feats.reshape(-1, 8).std(axis=0)
    m = bnos.Mlp()
    m.set_params(p32, mu, sd)
    f, pr = torch.from_numpy(feats).cuda(), torch.from_numpy(pairs).cuda()
    out = torch.empty((R, n), dtype=torch.float32, device="cuda")
    m.forward(f, out)
    for s in {0, R // 2, R - 1}:
        one = torch.empty((1, n), dtype=torch.float32, device="cuda")
        m.forward(f[s:s + 1].contiguous(), one)
        assert torch.equal(one[0], out[s])
        want = oracle.mlp_forward(oracle_params(p32), (feats[s].astype(np.float64) - mu) / sd)
        assert rel(out[s].cpu().numpy().astype(np.float64), want) <= 1e-2
    # one Adam step from zero moments: lr * g / (|g| + 1e-8), up to |g| = 1e-6 within 1% of lr, plus the
    # rounding of the weights; the epoch's visiting order moves a gradient by FP32 rounding only
    g = torch.empty(N_PARAM, dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float64, device="cuda")
    m.grad(f, pr, g, loss, eps=0.1)
    trace = torch.zeros(1, dtype=torch.float32, device="cuda")
    lr = 1e-3
    m.train(f, pr, 1, R, lr, 7, eps=0.1, loss_trace=trace)
    torch.cuda.synchronize()
    got = m.get_params()[0].astype(np.float64)
    gd = g.cpu().numpy().astype(np.float64)
    w0 = p32.astype(np.float64)
    big = np.abs(gd) > np.maximum(1e-6, 1e-5 * np.abs(gd).max())
    assert n == 2 or big.any()                       # (two nodes: the only pair has probability 1)
    want = w0 - lr * np.sign(gd)
    assert (np.abs(got - want)[big] <= 0.011 * lr + 2.0 ** -22 * np.abs(w0)[big]).all()
    assert abs(trace.item() - loss.item()) <= 1e-5 * abs(loss.item())
    # the BF16 copies follow the new weights
    m.forward(f, out)
    want = oracle.mlp_forward(oracle_params(m.get_params()[0]), (feats[0].astype(np.float64) - mu) / sd)
    assert rel(out[0].cpu().numpy().astype(np.float64), want) <= 1e-2
    m.free()
