"""Read-outs and checkpoints that go through the pinned staging (copies of
one slot, of many, and of several planes at a time) against the state they
were made from: populations written and read back bit for bit (rounded to
FP32 where they are stored so), densities equal to their sums, and reads
from several threads at once, of which one has the staging and the others
copy without it."""
import threading

import numpy as np
import pytest

from tests import workloads as W
from tests.test_gpu_field_form import make
from tests.test_gpu_parity import _capi

pytestmark = pytest.mark.gpu


def sim_of(capi, N, shape, precision, lattice):
    wl = W.random_droplet(N, shape, seed=3, lattice=lattice)
    mix = wl.gpu_mixture()
    s = capi.Simulation(mix, lattice, precision, wl.shape, wl.rho)
    s._mix = mix
    return s


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("N,shape,lattice", [(1, (7, 5), 0), (3, (61, 33), 0), (1, (1031, 517), 0),
                                             (4, (701, 640), 0), (2, (9, 8, 7), 1),
                                             (3, (65, 66, 67), 1), (1, (150, 70, 33), 1)])
def test_populations_round_trip(N, shape, lattice, precision):
    capi = _capi()
    s = sim_of(capi, N, shape, precision, lattice)
    Q = 19 if lattice else 9
    rng = np.random.default_rng(5)
    g = rng.uniform(0.5, 1.5, size=(N, Q, s.sites))
    s.write_populations(g, 12)
    want = g.copy()
    if precision:
        want[:, 1:] = want[:, 1:].astype(np.float32)
    assert np.array_equal(s.read_populations(), want)
    rho = s.read_moments(velocity=False)["rho"].reshape(N, -1)
    assert np.max(np.abs(rho / want.sum(axis=1) - 1)) <= 1e-14
    s.close()


@pytest.mark.parametrize("N,shape", [(1, (7, 5)), (2, (301, 300)), (3, (400, 320)),
                                     (3, (400, 340)), (4, (701, 640))])
def test_moments_by_part_size(N, shape):
    """rho and u that a kernel writes out (parts up to 2 MiB), that go through
    the ring, and one of each: densities equal to the sums of the
    populations, and the momentum of rho and u as the device sums it."""
    capi = _capi()
    s = sim_of(capi, N, shape, 0, 0)
    s.step_n(2)
    out = s.read_moments()
    g = s.read_populations()
    rho, u = out["rho"].reshape(N, -1), out["u"].reshape(2, -1)
    assert np.max(np.abs(rho / g.sum(axis=1) - 1)) <= 1e-14
    d = s.diagnostics()
    p = (rho.sum(axis=0) * u).sum(axis=1)
    scale = (rho.sum(axis=0) * np.abs(u)).sum()
    assert np.max(np.abs(p - d["momentum"][:2])) <= 1e-12 * scale
    assert out["status"] == 0
    s.close()


def test_reads_from_several_threads():
    capi = _capi()
    sims = [sim_of(capi, 3, (400, 300 + k), 0, 0) for k in range(4)]
    for s in sims:
        s.step_n(3)
    ref = [s.read_populations() for s in sims]
    got = [None] * len(sims)

    def read(k):
        for _ in range(5):
            got[k] = sims[k].read_populations()

    th = [threading.Thread(target=read, args=(k,)) for k in range(len(sims))]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for a, b in zip(ref, got):
        assert np.array_equal(a, b)
    for s in sims:
        s.close()
