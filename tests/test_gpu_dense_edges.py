"""Dense builds at the ends of what the library takes: results that are no numbers."""
import numpy as np
import pytest

from workloads import gue

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fl(require_gpu):
    from paper_1508_07621_amd import floquet
    floquet.node_times(1.0, 1)          # loads the library or raises
    return floquet


# A caller's interval is checked at the steps with the smallest and the largest weight of
# Hmod; the step between them here has its spectrum far outside through the commutator, and
# T_300 overflows there: inf - inf leaves no number in U_T
@pytest.mark.parametrize("n", [5, 64, 150])
def test_unitarity_of_no_numbers_is_reported(fl, n):
    print("[case] no numbers", n, flush=True)
    rng = np.random.default_rng(n)
    f = np.array([[-1.0, -1.0], [2e4, -2e4], [1.0, 1.0]])
    ctx = fl.FloquetContext(h0=gue(n, rng), hmod=gue(n, rng), T=3.0, M=3, f_nodes=f, e_min=-20.0,
                            e_max=20.0, L=300)
    U = ctx.build_ut().cpu().numpy()
    rep = ctx.last_report
    print("[case] unitarity", rep["unitarity_max"], rep["unitarity_fro"], flush=True)
    assert np.isnan(U).any()
    assert rep["diverged"] == 1 and np.isnan(rep["unitarity_max"])
