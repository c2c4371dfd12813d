"""The batched kernels where their path or their work division changes: a batch
with an angle that needs the general stage code (the whole batch then runs the
512-thread kernel), circuits with three passes per layer, circuits whose work
items hold several tiles, and one circuit alone.  Held to the single-circuit
gradient as in the batch's own test: the same arithmetic in another order of
the qubits, 2e-5 (complex64) and 1e-10 (complex128) of the largest component."""
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


@pytest.mark.parametrize("precision", ["c64", "c128"])
@pytest.mark.parametrize("sizes,big", [([(14, 3), (17, 2), (24, 2), (15, 5)], True),
                                       ([(24, 1), (14, 6), (23, 2)], False), ([(26, 1), (14, 1)], False),
                                       ([(18, 4)], False)])
def test_batch_paths(sizes, big, precision):
    from paper_2604_26423_amd import Batch, Simulator
    inst = [(workloads.complete_graph_tenths(n, 40 + i), p) for i, (n, p) in enumerate(sizes)]
    ang = [oracle.gate_angles(*oracle.ramp_midpoint(p, 0.5, 0.3 + 0.1 * i)) for i, (_, p) in enumerate(sizes)]
    if big:
        ang[1][1][0] = 2.4  # |cos(theta / 2)| < 1/2
    b = Batch(inst, precision)
    print(f"batch {sizes} {precision}", flush=True)
    e, gzz, gx = b.forward_grad([a[0] for a in ang], [a[1] for a in ang])
    for i, (w, _) in enumerate(inst):
        sim = Simulator(w, precision)
        es, szz, sx = sim.adjoint(*ang[i])
        sim.close()
        scale = max(np.abs(szz).max(), np.abs(sx).max())
        tol = 1e-10 if precision == "c128" else 2e-5
        assert abs(e[i] - es) <= tol * abs(es)
        assert np.abs(gzz[i] - szz).max() <= tol * scale and np.abs(gx[i] - sx).max() <= tol * scale
    b.close()
