"""The precision of the weight gradients' sums over the rows: up to 8192 rows
only the 16 rows of a tile are added in FP32, everything beyond in FP64.

Every 128 rows hold two tiles with errors of +B, four with errors of B / 2^20,
and two with errors of -B; the rows of the large tiles are one row, repeated,
so that their products are equal (16 bits, 20 when a tile adds them: exact,
however the matrix cores round).  The large tiles add up to zero, so the
gradients must be those of the rows between.  These
rows alone give the reference: half as many rows change every operand by an
exact factor of two, so only the sums differ.

Tolerance: 16 products added in FP32 are off by at most 16 2^-24 of the sum of
their magnitudes, in both runs; the norm of what the rows of a weight add up to
is above 2^-3 of that sum's (errors of one sign, inputs about 1): 2 * 16 * 2^-24 *
8 = 1.6e-5.  Added on in FP32 a large tile, 16 B, would
leave 2^-24 * 16 B = B / 2^20 at each step, a whole row's error.
"""
import numpy as np
import pytest
import torch

import paper_2201_10132_amd as P
from oracle import learned as L
from tests import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [128, 1024, 8192])
def test_cancelling_rows_leave_the_others_exact(n):
    nin, nout, chunks = 54, 5, n // 128
    print(f"mlp sums n={n}", flush=True)
    m = P.Mlp(nin, 64, nout, seed=11)

    def dev(a):
        return torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda")

    big = np.repeat(1.0 + inputs.normal(2, (chunks, 1, nin)), 32, axis=1)
    mid = 1.0 + inputs.normal(1, (chunks, 64, nin))
    X = dev(np.concatenate([big, mid, big], axis=1))
    Y = torch.zeros((chunks, 128, nout), dtype=torch.float32, device="cuda")
    m.forward(X.data_ptr(), Y.data_ptr(), n)
    T = Y.clone()
    T[:, :32] -= 2.0 ** 10  # errors that round to 2^10 as BF16 operands
    T[:, 96:] += 2.0 ** 10
    T[:, 32:96] -= dev(2.0 ** -10 * (1.0 + inputs.rng(3).random(size=(chunks, 64, nout))))
    dW, _ = m.grads(X.data_ptr(), T.data_ptr(), n)
    Xr, Tr = X[:, 32:96].contiguous(), T[:, 32:96].contiguous()
    ref, _ = m.grads(Xr.data_ptr(), Tr.data_ptr(), n // 2)
    got = L.unflatten(dW.astype(np.float64), nin, 64, nout)
    want = L.unflatten(0.5 * ref.astype(np.float64), nin, 64, nout)
    err = {k: np.linalg.norm(got[k] - want[k]) / np.linalg.norm(want[k])
           for k in ("W1", "W2", "W3")}
    print(f"  {err}", flush=True)
    assert max(err.values()) < 1.6e-5, err
    m.close()


@pytest.mark.parametrize("n,run", [(57376, 128), (122912, 256), (300032, 512)])
def test_many_rows_add_up_to_their_halves(n, run):
    """From 57345 rows on a run of 128 rows, of 256 from 122881 and more beyond
    is added in FP32.  The gradients are the means of the two halves' (scaled by
    an exact 1/2); tolerance as above with that run: 2 run 2^-24 8."""
    nin, nout, half = 54, 5, n // 2
    print(f"mlp halves n={n}", flush=True)
    m = P.Mlp(nin, 64, nout, seed=5)

    def dev(a):
        return torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda")

    X = dev(1.0 + inputs.normal(7, (n, nin)))
    T = torch.zeros((n, nout), dtype=torch.float32, device="cuda")
    m.forward(X.data_ptr(), T.data_ptr(), n)
    T -= dev(1.0 + inputs.rng(8).random(size=(n, nout)))
    dW, loss = m.grads(X.data_ptr(), T.data_ptr(), n)
    parts = [m.grads(X[i:i + half].data_ptr(), T[i:i + half].data_ptr(), half) for i in (0, half)]
    got = L.unflatten(dW.astype(np.float64), nin, 64, nout)
    want = L.unflatten(0.5 * sum(g.astype(np.float64) for g, _ in parts), nin, 64, nout)
    err = {k: np.linalg.norm(got[k] - want[k]) / np.linalg.norm(want[k]) for k in got}
    print(f"  {err}", flush=True)
    assert max(err.values()) < 2 * run * 2.0 ** -24 * 8, err
    assert abs(loss - 0.5 * sum(v for _, v in parts)) < 1e-6 * loss
    m.close()
