"""Many shots: small states, whose launches hold at most 2^26 threads and then go
round again; counts on both sides of those at which shots go from 16 lanes each
to one lane each and back, in every layout and precision.  Shots are integers
and must be the oracle's."""
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


def random_state(n, precision):
    from paper_2604_26423_amd import Simulator
    sim = Simulator(workloads.complete_graph_tenths(n, n), precision)
    gen = torch.Generator(device="cuda").manual_seed(n)
    v = torch.randn(1 << n, 2, generator=gen, device="cuda", dtype=torch.float64)
    v /= torch.linalg.vector_norm(v)
    sim.set_amplitudes(torch.view_as_complex(v))
    return sim


def test_small_state_more_shots_than_threads():
    shots = (1 << 26) + 1025
    sim = random_state(4, "c64")
    print(f"shots n=4 {shots}", flush=True)
    got = sim.sample(shots, 3, on_device=True).cpu().numpy().view(np.uint64)
    assert np.array_equal(got, oracle.sample(sim.amplitudes().cpu().numpy(), 3, shots))
    sim.close()


@pytest.mark.parametrize("precision", ["c64", "c128"])
@pytest.mark.parametrize("n", [13, 15, 16, 22])
@pytest.mark.parametrize("shots", [(1 << 17) - 1, (1 << 17) + 77, (1 << 19) - 3, (1 << 19) + 1, (1 << 22) + 300])
def test_shots_one_lane_each(n, shots, precision):
    sim = random_state(n, precision)
    print(f"shots n={n} {precision} {shots}", flush=True)
    got = sim.sample(shots, 11, on_device=True).cpu().numpy().view(np.uint64)
    assert np.array_equal(got, oracle.sample(sim.amplitudes().cpu().numpy(), 11, shots))
    sim.close()


@pytest.mark.parametrize("precision", ["c64", "c128"])
def test_symmetric_shots_one_lane_each(precision):
    from paper_2604_26423_amd import Simulator
    sim = Simulator(workloads.complete_graph_tenths(17, 5), precision, symmetric=True)
    sim.forward(*oracle.gate_angles(*oracle.ramp_midpoint(2, 0.6, 0.6)))
    half = sim.amplitudes().cpu().numpy()
    for shots in (1000, (1 << 18) + 9):
        got = sim.sample(shots, 4, on_device=True).cpu().numpy().view(np.uint64)
        assert np.array_equal(got, oracle.sample_sym(half, 17, 4, shots))
    sim.close()
