"""Diagnostics, observables and the batch's amplitudes and health from the
passes over (node, Q-range) items, against sums over the copied-out state:
one workgroup, ragged tiles, a remainder of Q-nodes, and lattices on both
sides of the observables' size rule; each storage form."""
import numpy as np
import pytest

import paper_2201_10132_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nq,precision", [
    (16, 16, 6, P.TPL_FP64), (5, 13, 6, P.TPL_FP64), (70, 9, 10, P.TPL_FP32),
    (72, 30, 16, P.TPL_BF16), (65, 33, 12, P.TPL_FP64), (512, 511, 6, P.TPL_FP32),
    (512, 513, 6, P.TPL_FP32), (512, 513, 6, P.TPL_FP64)])
def test_passes_over_psi_match_the_copied_state(nx, ny, nq, precision):
    print(f"observe {nx}x{ny} nq {nq} precision {precision}", flush=True)
    t = P.Tpl(nx, ny, 20.0, 0.5, 0.8, periods=max(1, ny // 128), nq=nq, pre_steps=20,
              precision=precision, autotune=0)
    t.init(seed=4, perturbation=1e-2)
    t.step(2)
    st, d, m = t.get_state(populations=False), t.diagnostics(), t.moments()
    psi, U, n = st["psi"], st["U"], nx * ny
    # sums of n (times nqd) terms in another order: n eps relative
    tol = max(1e-12, 4e-16 * n)
    assert d["min_psi"] == psi.min()
    assert np.isclose(d["mass_P"] + d["mass_S"], m[0].sum(), rtol=tol)
    dev = U - U.mean(axis=2, keepdims=True)
    amp = np.sqrt((dev ** 2).sum() / n) / t.query("u0")
    assert np.isclose(d["amplitude"], amp, rtol=1e-9) and d["amplitude"] == t.amplitude()
    assert np.array_equal(m[1:3], U)
    # psi-weighted trace of C against the diagnostics' mean square extension
    ps = psi.sum(axis=0)
    q2 = (ps * (m[4] + m[6])).sum() / ps.sum() * t.query("sigma") ** 2
    assert np.isclose(d["qrms"] * t.query("R"), np.sqrt(q2), rtol=tol)
    t.close()


@pytest.mark.parametrize("precision", [P.TPL_FP64, P.TPL_FP32])
def test_batch_passes_match_each_instance(precision):
    """Lattices of unlike sizes in one launch: amplitudes bit for bit the
    instances' own, and a NaN in the smallest one's last row flags it alone."""
    print(f"observe batch {precision}", flush=True)
    sizes = [(96, 40), (16, 6), (65, 33), (128, 128)]
    b = P.Batch([dict(nx=x, ny=y, Re=20.0, Wi=0.5, beta=0.8, periods=1, seed=i, perturbation=1e-2)
                 for i, (x, y) in enumerate(sizes)],
                precision=precision, nq=6, pre_steps=20, autotune=0)
    b.init()
    b.step(2)
    assert np.array_equal(b.amplitudes(), [b.instance(i).amplitude() for i in range(4)])
    st = b.instance(1).get_state()
    st["XS"][0, 5, 15] = np.nan
    b.instance(1).set_state(**st)
    b.step(1)
    assert list(b.status()) == [0, 1, 0, 0]
    a = b.amplitudes()
    assert np.isnan(a[1])
    assert np.array_equal(a[[0, 2, 3]], [b.instance(i).amplitude() for i in (0, 2, 3)])
    b.close()
