"""States whose squared amplitudes sum to 4 or more cannot be sampled: the sums
of q(x) = floor(|a_x|^2 2^62) leave 64 bits, whichever sum is the first to do so
(that of 64 amplitudes, of a block of 8192, of a chunk of 2^26 or of all
chunks), and also where the wrapped total is exactly 0.  No single amplitude
is large.  A norm just below 4 is sampled by the rule."""
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


# n, number of equal amplitudes, from which index on
SPREAD = [(1, 2, 0), (5, 32, 0), (5, 8, 16), (12, 4096, 0), (14, 64, 128), (14, 16, 8208), (14, 8192, 8192),
          (14, 16384, 0), (27, 1 << 26, 1 << 26), (27, 1 << 20, (1 << 26) - (1 << 19)), (27, 1 << 27, 0)]


@pytest.mark.parametrize("precision", ["c64", "c128"])
@pytest.mark.parametrize("n,count,first", SPREAD)
def test_norm_of_four_or_more(n, count, first, precision):
    from paper_2604_26423_amd import Simulator, qs
    if n == 27 and precision == "c128":
        pytest.skip("one precision at the size with two chunks")
    sim = Simulator(workloads.complete_graph_tenths(n, 3), precision)

    def state(norm):
        # |a|^2 = norm / count, a power of two for norm = 4: exact as (x, 0) or (x, x)
        each = norm / count
        real = torch.zeros(1 << n, 2, dtype=torch.float64, device="cuda")
        if np.log2(4 / count) % 2 == 0:
            real[first:first + count, 0] = each ** 0.5
        else:
            real[first:first + count] = (each / 2) ** 0.5
        sim.set_amplitudes(torch.view_as_complex(real))

    print(f"norm n={n} {precision} {count} amplitudes", flush=True)
    for norm in (4.0, 5.0, 8.0):
        state(norm)
        for on_device in (False, True):
            with pytest.raises(qs.QSError, match="too large") as ei:
                sim.sample(20, 7, on_device=on_device)
            assert ei.value.status == qs.QS_ERR_STATE
        with pytest.raises(qs.QSError, match="too large"):
            sim.sample(0, 7)
    state(3.9)
    shots = sim.sample(1000, 7)
    assert shots.min() >= first and shots.max() < first + count
    if n < 27:
        assert np.array_equal(shots, oracle.sample(sim.amplitudes().cpu().numpy(), 7, 1000))
    sim.close()
