"""The row-walking restriction (factors 2 and 4) at the edges of its split:
coarse widths around a wave's 64 columns, coarse heights around its eight
rows, the smallest lattices; factor 6 takes the general kernel.  Tolerance as
for the general kernel: 1e-13 (sums of at most 49 terms of one sign)."""
import pytest

import paper_2201_10132_amd as P
from oracle import learned as L
from tests.gpu_common import max_rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [2, 4, 6])
@pytest.mark.parametrize("nxc,nyc", [(4, 4), (63, 9), (64, 8), (65, 7), (130, 17)])
def test_restriction_edges(m, nxc, nyc):
    fine = P.Tpl(m * nxc, m * nyc, 25.0, 0.6, 0.7, periods=1, nq=4, pre_steps=10)
    coarse = P.Tpl(nxc, nyc, 25.0, 0.6, 0.7, periods=1, nq=4, pre_steps=0)
    print(f"restrict {m} {nxc}x{nyc}", flush=True)
    fine.init(seed=3, perturbation=1e-2)
    coarse.init(seed=0, perturbation=0.0)
    coarse.restrict_from(fine)
    got, f = coarse.get_state(), fine.get_state()
    for k in ("XS", "XP", "psi", "U"):
        assert max_rel(got[k], L.restrict(f[k], m)) < 1e-13, k
    fine.close()
    coarse.close()
