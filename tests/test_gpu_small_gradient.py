"""Gradients of the single-workgroup kernels (n <= 13 complex64, 12 complex128)
against the oracle's gate-by-gate adjoint, each of the two gradients relative to
its own largest component: 1e-4 (complex64) and 1e-10 (complex128), as in the
other gradient tests.  With a bound of that kind a gradient of zeros, one of the
opposite sign and one whose layers are shifted by one fail; the oracle's values
are held to that first.

35 layers exceed one launch (32), 24 layers of 200 to 400 cut values several
groups of tables; weights up to 400 leave the table to some sizes and not to
others, weights up to 20000 to none."""
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


def far(got, want, tol):
    return np.abs(got - want).max() > tol * np.abs(want).max()


@pytest.mark.parametrize("n,precision", [(2, "c64"), (5, "c128"), (6, "c64"), (7, "c64"), (8, "c128"), (9, "c64"),
                                         (10, "c128"), (11, "c64"), (12, "c64"), (12, "c128"), (13, "c64")])
@pytest.mark.parametrize("p,wmax", [(35, 11), (24, 11), (3, 40), (3, 150), (3, 400), (2, 20000)])
def test_small_gradients(n, precision, p, wmax):
    from paper_2604_26423_amd import Simulator
    w = np.random.default_rng(n + p).integers(1, wmax, size=n * (n - 1) // 2, dtype=np.int32)
    tzz, tx = workloads.random_angles(p, n, scale=1.5)
    tzz = tzz * (11 / wmax)
    tol = 1e-4 if precision == "c64" else 1e-10
    e_ref, gzz_ref, gx_ref = oracle.adjoint(n, w, tzz, tx)
    for ref in (gzz_ref, gx_ref):  # what the bound has to tell apart
        assert far(np.zeros(p), ref, tol) and far(-ref, ref, tol) and far(np.roll(ref, 1), ref, tol)
    sim = Simulator(w, precision)
    print(f"small gradient n={n} {precision} p={p} W={w.sum()}", flush=True)
    for mode in ("uncompute", "store"):
        e, gzz, gx = sim.adjoint(tzz, tx, mode=mode)
        err = [np.abs(g - r).max() / np.abs(r).max() for g, r in ((gzz, gzz_ref), (gx, gx_ref))]
        print(f"  {mode}: <C> rel {abs(e - e_ref) / e_ref:.1e}, gradients rel {err[0]:.1e} {err[1]:.1e}", flush=True)
        assert abs(e - e_ref) <= (1e-5 if precision == "c64" else 1e-12) * e_ref
        assert not far(gzz, gzz_ref, tol) and not far(gx, gx_ref, tol)
    sim.close()
