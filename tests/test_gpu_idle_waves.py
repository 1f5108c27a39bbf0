"""Workgroups of four tiles whose last one is not full, with rows that do not
fill their last tile or with whole rows, two arrays or in place: idle waves must
store nothing.  A state that repeats along x stays so bit for bit, so a lattice
and several of it side by side must agree.  And ragged BF16 row tiles with eight
Q-slices in the kernel of 64 nodes per wave."""
import numpy as np
import pytest

import paper_2201_10132_amd as P

pytestmark = pytest.mark.gpu

CASES = [  # nx, ny, copies, groups of the one / the many, precision, options
    # whole rows in place: 1021 to 1023 tiles, three to one idle waves; twice
    # as wide 2042 to 2046 (511 groups, even again)
    (64, 1021, 2, (4, 4), P.TPL_FP64, dict(nq=4, periods=4, inplace=1)),
    (64, 1022, 2, (4, 4), P.TPL_FP32, dict(nq=4, periods=4, inplace=1)),
    (64, 1023, 2, (4, 4), P.TPL_FP64, dict(nq=4, periods=4, inplace=1, spring_shift=1)),
    # row tiles of 48 (60) of 64 nodes: 933 to 935 tiles, 1866 to 1870 of 32 (56)
    (48, 933, 2, (4, 4), P.TPL_BF16, dict(nq=4, periods=4, qsplit=1)),
    (48, 934, 2, (4, 4), P.TPL_BF16, dict(nq=4, periods=4, qsplit=1, qe_model=2, tau_ratio_p=0.5)),
    (48, 935, 2, (4, 4), P.TPL_BF16, dict(nq=4, periods=4, qsplit=1)),
    (60, 935, 2, (4, 4), P.TPL_FP32, dict(nq=4, periods=4, qsplit=1, spring_shift=1)),
    # flat tiles: 250 x 238 = 930 with one slice
    (125, 238, 2, (0, 4), P.TPL_FP64, dict(nq=6, periods=1, qsplit=1)),
]


def _tiled(st, rep):
    return {k: np.tile(v, (1,) * (v.ndim - 1) + (rep,)) for k, v in st.items()}


@pytest.mark.parametrize("nx,ny,rep,groups,precision,option", CASES)
def test_idle_waves_store_nothing(nx, ny, rep, groups, precision, option):
    print(f"idle waves {nx}x{ny} x{rep} precision {precision} {option}", flush=True)
    kw = dict(pre_steps=10, precision=precision, **option)
    one, many = (P.Tpl(nx * r, ny, 20.0, 0.5, 0.8, **kw) for r in (1, rep))
    one.init(seed=3, perturbation=1e-2)
    many.init(seed=0, perturbation=0.0)
    st = one.get_state()
    one.set_state(**st)
    many.set_state(**_tiled(st, rep))
    one.step(6)
    many.step(6)
    assert (one.query("group_x_used"), many.query("group_x_used")) == groups
    a, b = _tiled(one.get_state(), rep), many.get_state()
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    assert np.array_equal(np.tile(one.moments(), (1, 1, rep)), many.moments())
    one.close()
    many.close()


@pytest.mark.parametrize("nx,ny,rep,nq,precision,option", [
    (112, 40, 4, 6, P.TPL_BF16, {}),                    # 70 flat tiles / 280: both wide
    (112, 40, 4, 6, P.TPL_FP32, dict(spring_shift=1)),
    (112, 33, 4, 6, P.TPL_BF16, {}),                    # 58: narrow / 231: wide
    (112, 70, 2, 12, P.TPL_BF16, dict(qe_model=2, tau_ratio_p=0.5)),  # 123 / 245
])
def test_ragged_rows_with_eight_slices(nx, ny, rep, nq, precision, option):
    print(f"eight slices {nx}x{ny} x{rep} nq {nq} precision {precision} {option}", flush=True)
    kw = dict(periods=1, nq=nq, pre_steps=10, qsplit=8, precision=precision, **option)
    one, many = (P.Tpl(nx * r, ny, 20.0, 0.5, 0.8, **kw) for r in (1, rep))
    one.init(seed=3, perturbation=1e-2)
    many.init(seed=0, perturbation=0.0)
    st = one.get_state()
    one.set_state(**st)
    many.set_state(**_tiled(st, rep))
    one.step(6)
    many.step(6)
    a, b = _tiled(one.get_state(), rep), many.get_state()
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    one.close()
    many.close()
