"""Workspace of the pruning network's batches: its size by shape and batch, and
the training steps on both sides of the batch from which a deep network's
gradients take the place of its activations."""
import ctypes as C

import pytest

from paper_2211_17028_amd import tn


def _sizes(n_in, width, depth, batch):
    npar, sb, wb = C.c_int64(), C.c_size_t(), C.c_size_t()
    tn._check(tn._mlp_lib().tn_mlp_sizes(C.byref(tn.tn_mlp_shape(n_in, width, depth)), batch, C.byref(npar),
                                         C.byref(sb), C.byref(wb)))
    return wb.value


@pytest.mark.parametrize("n_in,width,depth", [(36, 272, 3), (36, 272, 6), (36, 512, 8), (36, 1024, 16), (4096, 300, 5),
                                              (257, 64, 16), (36, 4096, 2), (36, 256, 5)])
def test_size_of_layer_by_layer_networks(n_in, width, depth):
    """Activations, normalized rows, two gradient buffers and a row's few more,
    plus at most 256 MB of kept gradients and 512 tiles of FP64 partials."""
    last = 0
    for batch in sorted([1, 63, 64, 1000, 4096, 32768, 61680, 61681, 61682, 65536, 65537, 65538, 1 << 18, 1 << 20]):
        ws = _sizes(n_in, width, depth, batch)
        two = 4 * batch * (n_in + depth * width + 2 * max(width, n_in) + 2)
        assert ws <= two + (256 << 20) + 512 * 64 * 65 * 8 + batch // 2 + 16384, (batch, ws, two)
        assert ws >= last                       # a workspace of a batch holds every smaller one
        last = ws


@pytest.mark.gpu
@pytest.mark.parametrize("n", [65536, 65537])
def test_steps_around_the_limit_of_kept_gradients(n):
    """36 -> 1024 x 3 -> 1: gradients in place from 65537 rows on.  Against the
    same network in float64."""
    import torch
    n_in, width, depth = 36, 1024, 3
    print("mlp kept gradients", n, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n)
    net = tn.MLP(n_in=n_in, width=width, depth=depth, seed=5, max_batch=n)
    x, t = (torch.randn(n, c, device="cuda", generator=gen) for c in (n_in, 1))
    w = torch.rand(n, 1, device="cuda", generator=gen) + 0.5
    P, d = net.n_params, n_in
    net.gradients(x, t, w)
    g = net.state[2 * d + P:2 * d + 2 * P].clone()
    p = net.state[2 * d:2 * d + P].double().requires_grad_()
    h, at = x.double(), 0
    for l in range(depth + 1):
        dout = 1 if l == depth else width
        weight = p[at:at + dout * h.shape[1]].view(dout, -1)
        at += weight.numel()
        h = torch.nn.functional.linear(h, weight, p[at:at + dout])
        at += dout
        h = h if l == depth else torch.relu(h)
    loss = (w.double() * (h - t.double()) ** 2).mean()
    loss.backward()
    # FP32 sums of up to 1024 terms in each of 4 layers and back: an error of about
    # layers x sqrt(terms) x 2^-24 x 10
    assert (g.double() - p.grad).norm() <= 1e-4 * p.grad.norm()
    assert abs(net.loss.item() - loss.item()) <= 1e-4 * loss.item()
    other = tn.MLP(n_in=n_in, width=width, depth=depth, seed=5, max_batch=n)
    net.adam(1e-3)
    other.train_step(x, t, w, lr=1e-3)
    assert torch.equal(net.state, other.state) and torch.equal(net.loss, other.loss)
