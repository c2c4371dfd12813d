"""A circuit's results do not depend on the circuits that share its batch, bit for
bit: alone, among circuits in tangent form, and next to one whose large mixer
angle needs the general stage code."""
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


def circuit(n, p, seed, large=False):
    tzz, tx = oracle.gate_angles(*oracle.ramp_midpoint(p, 0.6, 0.3 + 0.05 * seed))
    if large:
        tx[p // 2] = 2.4  # |cos(theta / 2)| < 1/2
    return workloads.complete_graph_tenths(n, seed), tzz, tx


def run(circuits, precision):
    from paper_2604_26423_amd import Batch
    b = Batch([(w, len(tzz)) for w, tzz, _ in circuits], precision)
    e, gzz, gx = b.forward_grad([c[1] for c in circuits], [c[2] for c in circuits])
    b.close()
    return [(e[i], gzz[i], gx[i]) for i in range(len(circuits))]


@pytest.mark.parametrize("precision", ["c64", "c128"])
@pytest.mark.parametrize("large", [False, True])
def test_results_do_not_depend_on_batch_mates(large, precision):
    mine = [circuit(14, 3, 1, large), circuit(18, 4, 2, large), circuit(24, 2, 3, large)]
    small = [circuit(16, 5, 4), circuit(20, 2, 5)]
    big = [circuit(15, 6, 6, True), circuit(19, 2, 7, True)]
    print(f"batch mates {precision} large={large}", flush=True)
    alone = [run([c], precision)[0] for c in mine]
    for mates in (small, big, small + big):
        got = run(mates[:1] + mine + mates[1:], precision)[1:4]
        for (e, gzz, gx), (e1, gzz1, gx1) in zip(got, alone):
            assert e == e1 and np.array_equal(gzz, gzz1) and np.array_equal(gx, gx1)
