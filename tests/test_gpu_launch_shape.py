"""The launch shape that a step reports (group_*_used, qsplit_used) is the one
it ran in: the default's groups of four tiles, one tile per workgroup without
the autotuner, the caller's shape, and a shape that the tuner timed; whichever
it is, the state is bit for bit the same."""
import numpy as np
import pytest

import paper_2201_10132_amd as P

pytestmark = pytest.mark.gpu

FOURS, ONE = (4, 1, 1), (0, 0, 0)


def _run(nx, ny, precision, steps=4, **kw):
    kw = dict(dict(periods=max(1, ny // 256), nq=4, pre_steps=10, precision=precision), **kw)
    t = P.Tpl(nx, ny, 20.0, 0.5, 0.8, **kw)
    t.init(seed=2, perturbation=1e-2)
    t.step(steps)
    used = tuple(int(t.query(k)) for k in ("group_x_used", "group_y_used", "group_sync_used"))
    st, tune = t.get_state(), t.query("tune_ms")
    t.close()
    return st, used, tune


@pytest.mark.parametrize("nx,ny,precision,option,default", [
    (256, 256, P.TPL_FP64, {}, FOURS),                       # 256 groups
    (192, 342, P.TPL_FP64, dict(inplace=1), ONE),            # 1026 tiles: 257 groups
    (64, 1022, P.TPL_FP64, dict(inplace=1), FOURS),          # the last group two tiles
    (111, 1200, P.TPL_FP32, {}, FOURS),                      # flat tiles, 2082
    (500, 300, P.TPL_FP32, dict(spring_shift=1), FOURS),     # row tiles
    (370, 400, P.TPL_FP32, {}, ONE),                         # 2313 uneven, planes on lines
    (450, 400, P.TPL_FP32, {}, FOURS),                       # 2813, even
    (121, 1211, P.TPL_BF16, {}, ONE),                        # 2422 row tiles, uneven
    (200, 700, P.TPL_BF16, {}, FOURS),                       # 2800 row tiles
    (87, 2060, P.TPL_BF16, {}, ONE),                         # 2801 flat tiles, even
    (250, 300, P.TPL_BF16, dict(qsplit=1), ONE),             # 1200 row tiles
    (250, 230, P.TPL_BF16, dict(qsplit=1), ONE),             # 920: 230 groups
    (250, 255, P.TPL_BF16, dict(qsplit=1), FOURS),           # 1020
])
def test_default_group_is_reported(nx, ny, precision, option, default):
    print(f"launch shape {nx}x{ny} precision {precision} {option}", flush=True)
    ref, used, tune = _run(nx, ny, precision, autotune=0, **option)
    assert used == ONE and tune == 0
    st, used, tune = _run(nx, ny, precision, **option)
    assert used == default and tune == 0
    for k in ref:
        assert np.array_equal(st[k], ref[k]), k


@pytest.mark.parametrize("nx,ny,precision,option", [
    (192, 704, P.TPL_FP32, {}),           # 2112 tiles, fours the default but no 4 x 1 group
    (256, 544, P.TPL_FP64, dict(inplace=1)),
])
def test_tuned_shape_is_reported(nx, ny, precision, option):
    print(f"tuned shape {nx}x{ny} precision {precision} {option}", flush=True)
    ref, used, _ = _run(nx, ny, precision, steps=30, autotune=0, **option)
    assert used == ONE
    st, used, tune = _run(nx, ny, precision, steps=30, **option)
    print(f"  tuned {used}, {tune:.2f} ms", flush=True)
    assert tune > 0
    admitted = {ONE, (2, 2, 1), FOURS} | ({(4, 2, 1)} if nx % 256 == 0 else set())
    assert used in admitted
    for k in ref:
        assert np.array_equal(st[k], ref[k]), k


@pytest.mark.parametrize("nx,ny,precision,qs", [
    (128, 128, P.TPL_FP64, 8),
    (256, 232, P.TPL_FP64, 4),  # 928 tiles, 232 groups of four: uneven
    (250, 238, P.TPL_FP64, 1),  # 930
    (250, 256, P.TPL_FP64, 1),  # 1000
    (256, 256, P.TPL_FP64, 1),
    (256, 257, P.TPL_FP64, 2),  # 257 groups
    (480, 248, P.TPL_FP64, 2),  # 1860, 465 groups
    (352, 352, P.TPL_FP64, 1),  # 1936
    (256, 256, P.TPL_FP32, 2),
    (320, 256, P.TPL_FP64, 2),
])
def test_batch_of_one_takes_the_slices_of_its_lattice(nx, ny, precision, qs):
    """Without the autotuner the number of Q-slices, and with it the order of
    the sums over Q, is that of a context of its own: the same bits."""
    print(f"batch of one {nx}x{ny} precision {precision}", flush=True)
    kw = dict(nq=6, pre_steps=10, autotune=0)
    b = P.Batch([dict(nx=nx, ny=ny, Re=20.0, Wi=0.5, beta=0.8, periods=1, seed=2,
                      perturbation=1e-2)], precision=precision, **kw)
    b.init()
    b.step(5)
    t = P.Tpl(nx, ny, 20.0, 0.5, 0.8, periods=1, precision=precision, **kw)
    t.init(seed=2, perturbation=1e-2)
    t.step(5)
    assert t.query("qsplit_used") == qs and b.query("qsplit_used") == qs
    sa, sb = b.instance(0).get_state(), t.get_state()
    for k in sa:
        assert np.array_equal(sa[k], sb[k]), k
    b.close()
    t.close()
