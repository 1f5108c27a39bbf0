"""A batch's health check and amplitudes with one stable instance, which the
passes take by value, and with two again: a batch of one, and a batch whose
other instances went unstable."""
import numpy as np
import pytest

import paper_2201_10132_amd as P

pytestmark = pytest.mark.gpu


def _batch(sizes, precision):
    b = P.Batch([dict(nx=x, ny=y, Re=20.0, Wi=0.5, beta=0.8, periods=1, seed=i, perturbation=1e-2)
                 for i, (x, y) in enumerate(sizes)],
                precision=precision, nq=6, pre_steps=20, autotune=0)
    b.init()
    b.step(2)
    return b


def _break(b, i):
    st = b.instance(i).get_state()
    st["XS"][0, -1, -1] = np.nan
    b.instance(i).set_state(**st)
    b.step(1)


@pytest.mark.parametrize("precision", [P.TPL_FP64, P.TPL_FP32])
def test_passes_with_one_stable_instance(precision):
    print(f"observe one {precision}", flush=True)
    b = _batch([(65, 33)], precision)
    assert list(b.status()) == [0]
    assert b.amplitudes()[0] == b.instance(0).amplitude()
    _break(b, 0)
    assert list(b.status()) == [1] and np.isnan(b.amplitudes()[0])
    b.close()
    b = _batch([(96, 40), (16, 6), (65, 33)], precision)
    _break(b, 1)
    assert list(b.status()) == [0, 1, 0]
    assert np.array_equal(b.amplitudes()[[0, 2]], [b.instance(i).amplitude() for i in (0, 2)])
    _break(b, 0)
    assert list(b.status()) == [1, 1, 0]
    b.step(1)
    a = b.amplitudes()
    assert np.isnan(a[:2]).all() and a[2] == b.instance(2).amplitude()
    b.close()
