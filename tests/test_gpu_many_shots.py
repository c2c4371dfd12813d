"""More shots than one round of a launch draws: small states, whose launches
hold at most 2^26 threads and then go round again.  Shots are integers and must
be the oracle's."""
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
