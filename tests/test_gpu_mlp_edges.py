"""The network's training pass and update at the edges of their split (chunks
of 128 nodes, at most 256 workgroups, 16-node tiles, odd input rows) against
the FP64 oracle.  Gradients: the bar of test_gpu_learned.py (8 BF16 roundings
per block norm, backward at the GPU's own outputs).  Update: a few FP32
roundings of theta and of the step, and the operand copies renewed with it
(the next forward pass uses them: the BF16 bound)."""
import numpy as np
import pytest
import torch

import paper_2201_10132_amd as P
from oracle import learned as L
from tests import inputs

pytestmark = pytest.mark.gpu
U_BF16 = 2.0 ** -8


def _dev(a):
    return torch.tensor(np.asarray(a, dtype=np.float32), device="cuda")


@pytest.mark.parametrize("n,nin,nout", [(1, 54, 5), (127, 54, 5), (129, 33, 9), (2050, 64, 16),
                                        (33000, 1, 1)])
def test_training_pass_edges(n, nin, nout):
    print(f"mlp edges n={n} {nin}->{nout}", flush=True)
    m = P.Mlp(nin, 64, nout, seed=n)
    theta = m.get_params().astype(np.float64)
    # targets off zero: a mean gradient that does not cancel over the nodes
    X, T = inputs.normal(n, (n, nin)), 1.0 + inputs.normal(n + 1, (n, nout), 0.5)
    Xd, Td = _dev(X), _dev(T)
    Yd = torch.zeros((n, nout), dtype=torch.float32, device="cuda")
    m.forward(Xd.data_ptr(), Yd.data_ptr(), n)
    Y, Tf = Yd.cpu().numpy().astype(np.float64), T.astype(np.float32).astype(np.float64)
    dW, loss = m.grads(Xd.data_ptr(), Td.data_ptr(), n)
    assert abs(loss - L.loss(Y, Tf)) < 1e-5 * L.loss(Y, Tf)
    p = L.unflatten(theta, nin, 64, nout)
    _, cache = L.forward(p, X.astype(np.float32).astype(np.float64))
    g = L.backward(p, cache, Y, Tf)
    got = L.unflatten(dW.astype(np.float64), nin, 64, nout)
    for k in g:
        assert np.linalg.norm(got[k] - g[k]) < 8 * U_BF16 * np.linalg.norm(g[k]), k
    # the update, from the library's own gradients
    m.train_step(Xd.data_ptr(), Td.data_ptr(), n, lr=1e-3)
    new = m.get_params()
    want, _, _ = L.adam(theta, dW.astype(np.float64), np.zeros_like(theta), np.zeros_like(theta),
                        1, lr=1e-3)
    assert np.abs(new - want).max() < 1e-6 * np.abs(theta).max() + 1e-7
    # its operand copies: another network with these parameters packs the same
    other = P.Mlp(nin, 64, nout, seed=0)
    other.set_params(new)
    Y2, Y3 = torch.zeros_like(Yd), torch.zeros_like(Yd)
    m.forward(Xd.data_ptr(), Y2.data_ptr(), n)
    other.forward(Xd.data_ptr(), Y3.data_ptr(), n)
    assert torch.equal(Y2, Y3)
    m.close()
    other.close()
