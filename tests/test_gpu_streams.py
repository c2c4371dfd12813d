"""Passes on both sides of the sizes at which they change between ordinary and
nontemporal access: states of 2 and 4 MB, 32 and 64 MB, 128 and 256 MB in each
precision.  Amplitudes of complex64 against complex128 within 1e-5, <C> within
1e-6 relative and gradients within 5e-6 of the largest, as in the other tests
of complex64; the mixer and cost layers applied one by one give the state of
the fused passes."""
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


@pytest.mark.parametrize("n", [17, 18, 19, 21, 22, 23, 24, 25])
def test_streamed_sizes(n):
    from paper_2604_26423_amd import Simulator
    w = workloads.complete_graph_tenths(n, 20 + n)
    tzz, tx = oracle.gate_angles(*oracle.ramp_midpoint(2, 0.6, 0.6))
    print(f"streams n={n}", flush=True)
    a, b = Simulator(w, "c64"), Simulator(w, "c128")
    ga, gb = a.adjoint(tzz, tx), b.adjoint(tzz, tx)
    scale = max(np.abs(gb[1]).max(), np.abs(gb[2]).max())
    assert max(np.abs(x - y).max() for x, y in zip(ga[1:], gb[1:])) <= 5e-6 * scale
    for sim in (a, b):
        e, nrm = sim.forward(tzz, tx)
        assert abs(e - gb[0]) <= (1e-6 if sim is a else 1e-12) * gb[0] and abs(nrm - 1) <= 1e-5
    ref = b.amplitudes()
    assert (a.amplitudes() - ref).abs().max().item() <= 1e-5
    a.init_plus()
    for z, x in zip(tzz, tx):
        a.apply_cost_layer(float(z))
        a.apply_mixer(float(x))
    assert (a.amplitudes() - ref).abs().max().item() <= 1e-5
    a.close()
    b.close()
