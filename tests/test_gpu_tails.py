"""Complex64 gradients at sizes whose reverse passes end in last windows of one
to five register bits (the compile-time tails of the 256-thread reverse
junction and of the reverse of a plain pass; n = 24 has three passes), in both
adjoint modes.  Up to n = 21 against the oracle's gate-by-gate adjoint, n = 24
against complex128.  Tolerances of the other complex64 gradient tests:
<C> 1e-6 relative, gradients 5e-6 (uncompute) and 1e-4 (store)."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("n", [15, 16, 17, 18, 19, 21, 22, 24])
def test_reverse_tails(n):
    from paper_2604_26423_amd import Simulator
    w = workloads.complete_graph_tenths(n, 40 + n)
    tzz, tx = oracle.gate_angles(*oracle.ramp_midpoint(2, 0.6, 0.6))
    print(f"tails n={n}", flush=True)
    if n <= 21:
        e_ref, rzz, rx = oracle.adjoint(n, w, tzz, tx)
    else:
        ref = Simulator(w, "c128")
        e_ref, rzz, rx = ref.adjoint(tzz, tx)
        ref.close()
    scale = max(np.abs(rzz).max(), np.abs(rx).max())
    sim = Simulator(w, "c64")
    for mode, tol in (("uncompute", 5e-6), ("store", 1e-4)):
        e, gzz, gx = sim.adjoint(tzz, tx, mode=mode)
        err = max(np.abs(gzz - rzz).max(), np.abs(gx - rx).max()) / scale
        print(f"  {mode}: <C> rel {abs(e - e_ref) / e_ref:.2e}, gradient rel {err:.2e}", flush=True)
        assert abs(e - e_ref) <= 1e-6 * abs(e_ref)
        assert err <= tol
    sim.close()
