"""Noisy trajectories whose Pauli frame moves in almost every layer, in some of
them, and hardly ever (the cut values of the two register layouts are reloaded
only when a layer starts from them), over more layers than one chunk of draws
(16), with one table entry per cut value and with tables of two levels (heavy
weights) or more.  Amplitudes and error counts against the oracle's own draws,
amplitudes within the 1e-5 (complex64) and 1e-12 (complex128) of the other
trajectory tests.  <C> is an FP64 sum over the very amplitudes that the call
writes out: within 2^n roundings, 1e-12, of the oracle's sum over them."""
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
@pytest.mark.parametrize("wmax", [11, 60, 400])
@pytest.mark.parametrize("n,p", [(2, 19), (3, 18), (4, 19), (6, 17), (8, 18), (9, 18), (10, 17), (11, 5), (12, 4)])
def test_moving_frames(n, p, wmax, precision):
    from paper_2604_26423_amd import Trajectories
    w = np.random.default_rng(3 * n + p).integers(1, wmax, size=n * (n - 1) // 2, dtype=np.int32)
    tzz, tx = workloads.random_angles(p, n, scale=0.9)
    tzz = tzz * (11 / wmax)
    diag = oracle.cost_diagonal(n, w)
    atol = 1e-5 if precision == "c64" else 1e-12
    tr = Trajectories(w, precision)
    print(f"frames n={n} p={p} W={w.sum()} {precision}", flush=True)
    for eps in (0.4, 1.0 / (len(w) + 1), 0.2 / (len(w) + 1)):
        out = tr.run(tzz, tx, eps, 9, 5, traj0=3, states=True)
        st, ne, e = out["states"].cpu().numpy(), out["nerr"].cpu().numpy(), out["exp_c"].cpu().numpy()
        for t in range(5):
            ref, rn = oracle.noisy_trajectory(n, w, tzz, tx, eps, 9, 3 + t)
            assert ne[t] == rn
            assert np.abs(st[t] - ref).max() <= atol
            e_ref = oracle.expect(st[t], diag)[0]
            assert abs(e[t] - e_ref) <= 1e-12 * e_ref
    tr.close()
