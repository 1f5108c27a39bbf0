"""Rows that do not fill their last 64-node tile, and workgroups of four
consecutive tiles: a state that repeats along x stays so bit for bit, so a
lattice and several of it side by side, which take another kernel or another
grouping, must agree bitwise."""
import numpy as np
import pytest

import paper_2201_10132_amd as P

pytestmark = pytest.mark.gpu

CASES = [  # nx, ny, copies, precision, Q-slices, options
    (48, 21, 4, P.TPL_BF16, 1, {}),                       # one tile a row, 21 % 4 idle waves
    (96, 7, 2, P.TPL_BF16, 1, dict(qe_model=2, tau_ratio_p=0.5)),
    (96, 7, 2, P.TPL_BF16, 4, {}),
    (112, 5, 4, P.TPL_BF16, 8, dict(nq=6)),               # narrow kernel / wide one
    (112, 5, 4, P.TPL_FP32, 1, {}),
    (112, 5, 4, P.TPL_FP32, 1, dict(qe_model=2, tau_ratio_p=0.5)),
    (112, 6, 4, P.TPL_FP32, 1, dict(spring_shift=1)),
    (112, 6, 4, P.TPL_FP32, 4, dict(spring_shift=1)),
    (80, 6, 4, P.TPL_FP32, 1, dict(spring_shift=1)),      # flat: too many idle lanes
    (85, 253, 3, P.TPL_FP64, 1, dict(nq=4, periods=2)),   # 337 tiles / 1009 in fours
    (111, 400, 3, P.TPL_FP32, 1, dict(nq=4, periods=4)),  # 694 tiles / 2082 in fours
    (64, 255, 4, P.TPL_FP64, 1, dict(nq=4, periods=2, inplace=1)),  # 255 / 1020
]


@pytest.mark.parametrize("nx,ny,rep,precision,qs,option", CASES)
def test_ragged_rows_are_bitwise_whole_rows(nx, ny, rep, precision, qs, option):
    print(f"ragged rows {nx}x{ny} x{rep} precision {precision} qs {qs} {option}", flush=True)
    kw = dict(dict(periods=1, nq=6, pre_steps=20, qsplit=qs, precision=precision, autotune=0),
              **option)
    one = P.Tpl(nx, ny, 20.0, 0.5, 0.8, **kw)
    many = P.Tpl(nx * rep, ny, 20.0, 0.5, 0.8, **kw)
    one.init(seed=3, perturbation=1e-2)
    many.init(seed=0, perturbation=0.0)
    st = one.get_state()
    one.set_state(**st)
    many.set_state(**{k: np.tile(v, (1,) * (v.ndim - 1) + (rep,)) for k, v in st.items()})
    one.step(6)
    many.step(6)
    a, b = one.get_state(), many.get_state()
    for k in a:
        assert np.array_equal(np.tile(a[k], (1,) * (a[k].ndim - 1) + (rep,)), b[k]), k
    one.close()
    many.close()
