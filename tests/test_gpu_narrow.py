"""The step kernel for few nodes (lanes are (node, Q-node) pairs, 16 or 4
nodes per workgroup): parity with the oracle at the edges of its split, and
bitwise equality with the 64-nodes-per-wave kernel at eight Q-slices, which
sums in the same order.

Tolerances: against the oracle as for any one step from a random state
(tests/test_gpu_parity.py): 1e-14, and 1e-13 after 20 steps.
"""
import numpy as np
import pytest

import paper_2201_10132_amd as P
from tests.gpu_common import compare_states, make_pair, max_rel
from tests.test_gpu_parity import _random_state

pytestmark = pytest.mark.gpu

# 16 nodes per workgroup hold 32 Q-nodes per pass, 4 nodes 128 (FP64, up to
# 1024 nodes, more than 32 Q-nodes).
CASES = [
    dict(nx=5, ny=7, nq=4, periods=1),                   # 12 Q-nodes: a part of one pass
    dict(nx=16, ny=16, nq=6, periods=1),                 # 32 Q-nodes: exactly one pass
    dict(nx=1, ny=37, nq=8, periods=2),                  # a column, 4 nodes, ragged
    dict(nx=13, ny=9, nq=16, periods=1),                 # 4 nodes, two passes, ragged
    dict(nx=32, ny=32, nq=8, periods=1),                 # 1024 nodes: the last with 4
    dict(nx=41, ny=25, nq=8, periods=1),                 # 1025 nodes: 16, ragged, two passes
    dict(nx=48, ny=40, nq=12, periods=1, spring=1),      # four passes
    dict(nx=70, ny=20, nq=10, periods=1, spring_shift=1),
    dict(nx=70, ny=20, nq=10, periods=1, qe_model=2, tau_ratio_p=0.5),
    dict(nx=24, ny=20, nq=10, periods=1, gradients=1),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c['nx']}x{c['ny']}q{c['nq']}")
def test_narrow_step_parity(case):
    c = dict(case)
    nx, ny = c.pop("nx"), c.pop("ny")
    t, o = make_pair(nx, ny, 20.0, 0.5, 0.8, c.pop("periods"), qsplit=8, pre_steps=0, **c)
    print(f"narrow {case}", flush=True)
    t.init(seed=0, perturbation=0.0)
    st = _random_state(t.nqd, ny, nx, o, seed=3)
    t.set_state(**st)
    o.set_state(**st)
    t.step(1); o.step(1)
    compare_states(t.get_state(), o.get_state(), 1e-14)
    t.step(19); o.step(19)
    compare_states(t.get_state(), o.get_state(), 1e-13)
    assert max_rel(t.moments(), o.observables()) < 1e-13


@pytest.mark.parametrize("precision", [P.TPL_FP64, P.TPL_FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("option", [{}, dict(spring_shift=1), dict(qe_model=2, tau_ratio_p=0.5)],
                         ids=["taylor", "shift", "model2"])
def test_narrow_is_bitwise_the_wide_kernel(precision, option):
    """A batch of more than 128 tiles takes the 64-node kernel, its instances
    alone the narrow one (base-state columns: the batch's too)."""
    insts = [dict(nx=16, ny=16, Re=20.0, Wi=0.5, beta=0.8, periods=1, seed=1, perturbation=1e-2),
             dict(nx=13, ny=9, Re=12.0, Wi=0.4, beta=0.9, periods=1, seed=3, perturbation=1e-2),
             dict(nx=70, ny=24, Re=30.0, Wi=0.5, beta=0.8, periods=2, seed=2, perturbation=1e-2),
             dict(nx=120, ny=72, Re=40.0, Wi=1.0, beta=0.7, periods=1, seed=4, perturbation=1e-2)]
    print(f"narrow vs wide {precision} {option}", flush=True)
    kw = dict(nq=8, pre_steps=40, qsplit=8, **option)
    b = P.Batch(insts, precision=precision, autotune=0, graph_steps=0, **kw)
    b.init()
    assert b.query("items") > 128 and b.query("qsplit_used") == 8
    b.step(6)
    for i, d in enumerate(insts[:3]):
        t = P.Tpl(d["nx"], d["ny"], d["Re"], d["Wi"], d["beta"], periods=d["periods"],
                  precision=precision, autotune=0, **kw)
        t.init(seed=d["seed"], perturbation=d["perturbation"])
        t.step(6)
        assert t.query("qsplit_used") == 8
        sa, sb = b.instance(i).get_state(), t.get_state()
        for k in sa:
            assert np.array_equal(sa[k], sb[k]), (i, k)
        assert np.array_equal(b.instance(i).moments(), t.moments()), i
        t.close()
    b.close()


@pytest.mark.parametrize("precision", [P.TPL_FP64, P.TPL_FP32, P.TPL_BF16],
                         ids=["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("nq,option", [(6, {}), (12, {}), (12, dict(qe_model=2, tau_ratio_p=0.5))],
                         ids=["nq6", "nq12", "nq12model2"])
def test_narrow_is_bitwise_the_wide_kernel_on_a_repeated_state(precision, nq, option):
    """A state that repeats along x stays so, bit for bit: the 64 x 40 lattice
    takes the narrow kernel, three or four of it side by side the wide one."""
    print(f"narrow vs wide repeated {precision} nq={nq} {option}", flush=True)
    kw = dict(periods=1, nq=nq, pre_steps=30, qsplit=8, precision=precision, autotune=0, **option)
    rep = 3 if nq == 6 else 4
    one = P.Tpl(64, 40, 20.0, 0.5, 0.8, **kw)
    many = P.Tpl(64 * rep, 40, 20.0, 0.5, 0.8, **kw)
    one.init(seed=2, perturbation=1e-2)
    many.init(seed=0, perturbation=0.0)
    st = one.get_state()
    one.set_state(**st)
    many.set_state(**{k: np.tile(v, (1,) * (v.ndim - 1) + (rep,)) for k, v in st.items()})
    one.step(5)
    many.step(5)
    a, b = one.get_state(), many.get_state()
    for k in a:
        assert np.array_equal(np.tile(a[k], (1,) * (a[k].ndim - 1) + (rep,)), b[k]), k
    one.close()
    many.close()
