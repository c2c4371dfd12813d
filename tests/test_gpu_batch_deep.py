"""A batch so deep that its partial sums (2^21 rows at most wait together) are
reduced in several groups of rounds: two circuits of 22 qubits in complex128,
1024 rows per summed step, 1100 and 1000 layers.  Held to the single-circuit
gradient as in the batch's own test, 1e-10 of the largest component."""
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


def test_sums_in_groups():
    from paper_2604_26423_amd import Batch, Simulator
    n, depths = 22, (1100, 1000)
    assert sum(1024 * (p + 1) for p in depths) > 1 << 21
    inst = [(workloads.complete_graph_tenths(n, 70 + i), p) for i, p in enumerate(depths)]
    ang = [oracle.gate_angles(*oracle.ramp_midpoint(p, 0.5, 0.4)) for p in depths]
    print(f"deep batch n={n} p={depths}", flush=True)
    b = Batch(inst, "c128")
    e, gzz, gx = b.forward_grad([a[0] for a in ang], [a[1] for a in ang])
    b.close()
    for i, (w, _) in enumerate(inst):
        sim = Simulator(w, "c128")
        es, szz, sx = sim.adjoint(*ang[i])
        sim.close()
        scale = max(np.abs(szz).max(), np.abs(sx).max())
        assert abs(e[i] - es) <= 1e-10 * abs(es)
        assert np.abs(gzz[i] - szz).max() <= 1e-10 * scale and np.abs(gx[i] - sx).max() <= 1e-10 * scale
