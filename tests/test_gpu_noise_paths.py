"""Noisy trajectories where the kernel changes its path: cut values too many for
one table entry each (528 of them and more), one layer more than a chunk of
draws, graphs of every layout (n = 2 and 3 without middle qubits, 4 to 12 with
up to four), an odd and an even number of layers.  Amplitudes, error counts and
<C> against the oracle's own draws, within the tolerances of the other
trajectory tests: amplitudes 1e-5 (complex64) and 1e-12 (complex128), <C> 1e-6
and 1e-12 relative."""
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
@pytest.mark.parametrize("n,p,wmax", [(2, 3, 11), (3, 2, 11), (4, 17, 11), (7, 2, 11), (8, 3, 11), (9, 2, 11),
                                      (10, 17, 11), (10, 2, 40), (11, 3, 11), (12, 2, 17), (12, 16, 11)])
def test_noise_paths(n, p, wmax, precision):
    from paper_2604_26423_amd import Trajectories
    w = np.random.default_rng(n + p).integers(1, wmax, size=n * (n - 1) // 2, dtype=np.int32)
    if wmax > 11:
        assert 528 <= w.sum() < 8192 // 3
    tzz, tx = workloads.random_angles(p, n, scale=0.9)
    print(f"noise n={n} p={p} W={w.sum()} {precision}", flush=True)
    tr = Trajectories(w, precision)
    out = tr.run(tzz, tx, 0.03, 5, 6, traj0=2, states=True)
    st, ne, e = out["states"].cpu().numpy(), out["nerr"].cpu().numpy(), out["exp_c"].cpu().numpy()
    atol, rtol = (1e-5, 1e-6) if precision == "c64" else (1e-12, 1e-12)
    diag = oracle.cost_diagonal(n, w)
    for t in range(6):
        ref, rn = oracle.noisy_trajectory(n, w, tzz, tx, 0.03, 5, 2 + t)
        assert ne[t] == rn
        assert np.abs(st[t] - ref).max() <= atol
        e_ref = oracle.expect(ref, diag)[0]
        assert abs(e[t] - e_ref) <= rtol * e_ref
    tr.close()
