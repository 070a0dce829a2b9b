"""Scores written over the network's own inputs: tn_mlp_forward with d_y inside
d_x or inside the workspace gives the values of a separate output, on the
whole-network launch and layer by layer."""
import ctypes as C

import numpy as np
import pytest

from paper_2211_17028_amd import tn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_in,width,depth,n", [(36, 128, 3, 4096), (1, 16, 1, 100), (5, 33, 2, 16400),   # one launch
                                                (36, 272, 1, 700), (257, 64, 2, 130)])                    # layers
@pytest.mark.parametrize("where", ["x_head", "x_tail", "ws_head", "ws_output", "ws_middle"])
def test_outputs_over_the_inputs(n_in, width, depth, n, where):
    import torch
    print("mlp overlap", n_in, width, depth, n, where, flush=True)
    rng = np.random.default_rng([n_in, width, n])
    net = tn.MLP(n_in=n_in, width=width, depth=depth, seed=3, max_batch=n)
    x = torch.from_numpy(rng.standard_normal((n, n_in)).astype(np.float32)).cuda()
    want = net.forward(x)
    flat = x.view(-1)
    up = lambda v: (v + 63) // 64 * 64                                        # noqa: E731
    at = up(up(n * n_in) + depth * n * width)                                  # the workspace's own output array
    y = {"x_head": flat[:n], "x_tail": flat[-n:], "ws_head": net.ws[:n], "ws_output": net.ws[at + 1:at + 1 + n],
         "ws_middle": net.ws[at - n:at]}[where]
    ptr = lambda t: C.c_void_p(t.data_ptr())                                   # noqa: E731
    tn._check(tn._mlp_lib().tn_mlp_forward(C.byref(net.shape), ptr(net.state), ptr(x), n, ptr(y), ptr(net.ws), None))
    torch.cuda.synchronize()
    assert torch.equal(y, want)
