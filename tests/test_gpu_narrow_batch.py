"""The batched step for few nodes: a batch of at most 64 tiles with eight
Q-slices takes it, the same instances with a larger one beside them the kernel
of 64 nodes per wave; both must give the contexts' own states bit for bit."""
import numpy as np
import pytest

import paper_2201_10132_amd as P

pytestmark = pytest.mark.gpu

ROWS = [dict(nx=16, ny=16, Re=20.0, Wi=0.5, beta=0.8, periods=1, seed=1, perturbation=1e-2),
        dict(nx=13, ny=9, Re=12.0, Wi=0.4, beta=0.9, periods=1, seed=3, perturbation=1e-2),
        dict(nx=70, ny=24, Re=30.0, Wi=0.5, beta=0.8, periods=2, seed=2, perturbation=1e-2),
        dict(nx=120, ny=72, Re=40.0, Wi=1.0, beta=0.7, periods=1, seed=4, perturbation=1e-2)]


def _states(rows, precision, items, **kw):
    b = P.Batch(rows, precision=precision, autotune=0, graph_steps=0, **kw)
    b.init()
    assert b.query("qsplit_used") == 8 and items(b.query("items"))
    b.step(6)
    out = [(b.instance(i).get_state(), b.instance(i).moments()) for i in range(len(rows))]
    b.close()
    return out


@pytest.mark.parametrize("precision", [P.TPL_FP64, P.TPL_FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("option", [{}, dict(spring_shift=1), dict(qe_model=2, tau_ratio_p=0.5)],
                         ids=["taylor", "shift", "model2"])
@pytest.mark.parametrize("few", [3, 2], ids=["33tiles", "6tiles"])
def test_narrow_batch_is_bitwise_the_wide_one_and_the_contexts(few, precision, option):
    """33 tiles: 16 nodes per workgroup; 6 tiles (less than 1024 nodes, more
    than 32 Q-nodes): 4 in FP64."""
    print(f"narrow batch of {few} {precision} {option}", flush=True)
    kw = dict(nq=8, pre_steps=40, qsplit=8, **option)
    small = _states(ROWS[:few], precision, lambda n: n <= (16 if few == 2 else 64), **kw)
    large = _states(ROWS, precision, lambda n: n > 128, **kw)
    for i, d in enumerate(ROWS[:few]):
        t = P.Tpl(d["nx"], d["ny"], d["Re"], d["Wi"], d["beta"], periods=d["periods"],
                  precision=precision, autotune=0, **kw)
        t.init(seed=d["seed"], perturbation=d["perturbation"])
        t.step(6)
        own = (t.get_state(), t.moments())
        t.close()
        for st, m in (small[i], large[i]):
            for k in st:
                assert np.array_equal(st[k], own[0][k]), (i, k)
            assert np.array_equal(m, own[1]), i
