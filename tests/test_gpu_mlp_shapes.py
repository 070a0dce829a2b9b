"""GPU tests of the pruning network's kernels at the edges of their launches:
rows and columns around the row blocks and matrix-core tiles, and shapes on
both sides of the rule that chooses between the whole-network launch and the
layer-by-layer one, against the FP64 reference network."""
import numpy as np
import pytest

from oracle import mlp as omlp
from paper_2211_17028_amd import tn

pytestmark = pytest.mark.gpu

# FP32 sums of up to 272 terms in each of up to 6 layers (and back): an error of
# about layers x sqrt(terms) x 2^-24 x 10 for cancellation, under 1e-4 of the result
TOL = 1e-4


@pytest.mark.parametrize("n_in,width,depth,n", [
    (36, 128, 3, 1), (36, 128, 3, 15), (36, 128, 3, 17), (36, 128, 2, 1000), (5, 33, 1, 63), (1, 1, 1, 64),
    (3, 17, 5, 130), (256, 256, 2, 300), (36, 144, 4, 129), (130, 96, 1, 65),      # one launch
    (36, 32, 1, 8200), (36, 32, 2, 16400),                                         # more rows per block
    (257, 64, 2, 70), (36, 272, 1, 100), (36, 256, 5, 40),                         # layer by layer
])
def test_forward_gradients_and_step(n_in, width, depth, n):
    import torch
    print("mlp", n_in, width, depth, n, flush=True)
    rng = np.random.default_rng([n_in, width, depth, n])
    net = tn.MLP(n_in=n_in, width=width, depth=depth, seed=7, max_batch=n)
    x = rng.standard_normal((n, n_in)).astype(np.float32) * 2 - 1
    t, w = rng.standard_normal(n).astype(np.float32), rng.uniform(0.5, 2.0, n).astype(np.float32)
    xd, td, wd = (torch.from_numpy(a).cuda() for a in (x, t, w))
    P, d = net.n_params, n_in
    net.state[:d] = torch.from_numpy(rng.standard_normal(d).astype(np.float32)).cuda()
    net.state[d:2 * d] = torch.from_numpy(rng.uniform(0.5, 1.5, d).astype(np.float32)).cuda()
    net.state[2 * d:2 * d + P] += 0.01
    st = net.state.cpu().numpy().astype(np.float64)
    y_ref = omlp.forward(st, x, n_in, width, depth)[0]
    y = net.forward(xd)
    assert np.linalg.norm(y.cpu().numpy() - y_ref) <= TOL * np.linalg.norm(y_ref)
    assert torch.equal(y, net.forward(xd))
    for weights, wt in ((w, wd), (np.ones(n, np.float32), None)):
        net.gradients(xd, td, wt)
        g = net.state[2 * d + P:2 * d + 2 * P].clone()
        g_ref = omlp.gradients(st, x, t, weights, n_in, width, depth)
        assert np.linalg.norm(g.cpu().numpy() - g_ref) <= TOL * np.linalg.norm(g_ref)
        loss_ref = omlp.loss(st, x, t, weights, n_in, width, depth)
        assert abs(net.loss.item() - loss_ref) <= TOL * loss_ref
        net.gradients(xd, td, wt)
        assert torch.equal(g, net.state[2 * d + P:2 * d + 2 * P])
    # a training step is the gradients followed by the update, bit for bit
    other = tn.MLP(n_in=n_in, width=width, depth=depth, seed=7, max_batch=n)
    other.state.copy_(net.state)
    net.gradients(xd, td, None)
    net.adam(1e-3)
    other.train_step(xd, td, lr=1e-3)
    assert torch.equal(net.state, other.state) and torch.equal(net.loss, other.loss)
