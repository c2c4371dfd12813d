"""The readouts where their work division changes, on a state set by hand:
shots below and above the counts where a workgroup takes several rounds, states
of one block, one chunk and several chunks; <C> and the norm for states below
and above one workgroup's stride; histograms of one bin, of a ragged number of
bins and of bins beyond the pinned buffer.  Shots and masses are integers and
must be the oracle's; <C> is an FP64 sum: within 1e-13."""
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
    from paper_2604_26423_amd import qs
    qs.lib()


def random_state(n, precision, seed):
    from paper_2604_26423_amd import Simulator
    sim = Simulator(workloads.complete_graph_tenths(n, seed), precision)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    v = torch.randn(1 << n, 2, generator=gen, device="cuda", dtype=torch.float64)
    v /= torch.linalg.vector_norm(v)
    sim.set_amplitudes(torch.view_as_complex(v))
    return sim


@pytest.mark.parametrize("precision", ["c64", "c128"])
@pytest.mark.parametrize("n,shots", [(1, 3), (12, 1024), (12, 1025), (13, 15), (13, 17), (14, 1), (18, (1 << 19) + 5),
                                     (27, 70000)])
def test_shots(n, shots, precision):
    if n == 27 and precision == "c128":
        pytest.skip("one precision at the size with two chunks")
    sim = random_state(n, precision, n)
    psi = sim.amplitudes().cpu().numpy()
    print(f"shots n={n} {precision} {shots}", flush=True)
    assert np.array_equal(sim.sample(shots, 11), oracle.sample(psi, 11, shots))
    assert np.array_equal(sim.sample(shots, 11, on_device=True).cpu().numpy().view(np.uint64),
                          oracle.sample(psi, 11, shots))
    sim.close()


def test_no_shots_still_reports_an_empty_state():
    from paper_2604_26423_amd import qs
    for n in (5, 15):
        sim = random_state(n, "c64", 1)
        assert len(sim.sample(0, 1)) == 0
        sim.set_amplitudes(torch.zeros(1 << n, dtype=torch.complex64, device="cuda"))
        with pytest.raises(qs.QSError) as ei:
            sim.sample(0, 1)
        assert ei.value.status == qs.QS_ERR_STATE
        sim.close()


@pytest.mark.parametrize("precision", ["c64", "c128"])
@pytest.mark.parametrize("n", [1, 2, 9, 10, 11, 19, 22])
def test_expect(n, precision):
    sim = random_state(n, precision, n)
    e_ref, n_ref = oracle.expect(sim.amplitudes().cpu().numpy(), oracle.cost_diagonal(n, sim.w))
    e, norm = sim.expect()
    assert abs(e - e_ref) <= 1e-13 * max(e_ref, 1) and abs(norm - n_ref) <= 1e-13
    sim.close()


@pytest.mark.parametrize("n,nbins", [(1, 1), (11, 31), (11, 33), (16, 1), (16, 8192), (16, 8193), (16, 200000)])
def test_histogram(n, nbins):
    from paper_2604_26423_amd import qs
    sim = random_state(n, "c64", n)
    want = oracle.cost_histogram(sim.amplitudes().cpu().numpy(), oracle.cost_diagonal(n, sim.w), nbins)
    assert np.array_equal(qs.qs_cost_histogram(sim.handle, sim.diag, nbins), want)
    out = torch.empty(nbins, dtype=torch.int64, device="cuda")
    assert np.array_equal(qs.qs_cost_histogram(sim.handle, sim.diag, nbins, out).cpu().numpy().view(np.uint64), want)
    sim.close()
