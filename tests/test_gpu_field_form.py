"""Runs of steps in field form (D2Q9 at tau = 1: populations read at a run's
start and written at its end, only rho_i, j and s between the steps) against
the fused kernels, which keep them in memory at every step.

Both add up the same rounded populations in the same order, so the bar is
bitwise, over widths either side of the 60-column strips, heights either
side of the rows per item, component counts 1 ... 10, run lengths that use
plain launches, a captured graph and both, runs continued from either
population buffer, and batches.  The grids are large enough for the
autotuner to take the field form.  The same on D3Q19 against the multi-pass
kernels.
"""
import numpy as np
import pytest

from tests import workloads as W
from tests.test_gpu_parity import _capi

pytestmark = pytest.mark.gpu


def make(capi, wl, precision, kernel=0, rows=0):
    mix = wl.gpu_mixture()
    s = capi.Simulation(mix, 0, precision, wl.shape, wl.rho)
    s._mix = mix
    if kernel:
        s.set_tuning(kernel, rows)
    return s


def field(N, shape, seed):
    """N = 1: a C1 slab; up to 4: a drop; more components: the first N of the
    ten-component field's mixture, uniform with noise (the oracle advances
    each over these runs without leaving the EOS domain)."""
    if N == 1:
        from inputs import fields as Fi
        wl = W.vle(1, *shape)
        wl.rho = Fi.add_noise(wl.rho, 1e-3, seed)
        return wl
    if N <= 4:
        return W.random_droplet(N, shape, seed=seed)
    from inputs import components as C, fields as Fi
    st = W.states()["spinodal10"]
    rho = Fi.add_noise(Fi.uniform(shape[0], shape[1], st["rho_uniform"][:N]), 1e-2, seed)
    return W.Workload(C.N_ALKANES[:N], 325.0, rho, shape, kij=np.array(st["kij"])[:N, :N])


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("N,shape,seed", [
    (1, (1021, 1019), 9), (1, (512, 511), 9), (2, (541, 600), 11), (3, (479, 361), 31), (4, (659, 240), 11),
    (6, (361, 181), 4), (9, (239, 211), 4), (10, (181, 300), 4), (10, (420, 97), 5)])
def test_field_form_matches_fused_bitwise(N, shape, seed, precision):
    capi = _capi()
    wl = field(N, shape, seed)
    a = make(capi, wl, precision, 2, 16)
    b = make(capi, wl, precision)
    for n in (9, 1, 40, 101):         # one step swaps the buffers (fused)
        a.step_n(n)
        b.step_n(n)
        assert np.array_equal(a.read_populations(), b.read_populations()), n
        assert b.diagnostics()["status"] == 0
    a.close()
    b.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_field_form_large_batch_matches_alone_bitwise(precision):
    """Enough rows for the step by single wavefronts to be the faster one."""
    capi = _capi()
    wls = [W.random_droplet(3, s, seed=31) for s in ((301, 240), (256, 256), (61, 400), (119, 121),
                                                     (180, 7))] * 4
    ref = [make(capi, wl, precision, 3, 5) for wl in wls[:5]]
    got = [make(capi, wl, precision) for wl in wls]
    for n in (12, 70):
        for s in ref:
            s.step_n(n)
        capi.step_many(got, n)
        for k, b in enumerate(got):
            assert np.array_equal(ref[k % 5].read_populations(), b.read_populations()), (n, k)
    for s in ref + got:
        s.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_field_form_batch_matches_alone_bitwise(precision):
    capi = _capi()
    wls = [W.random_droplet(3, s, seed=31) for s in ((301, 240), (59, 33), (61, 400), (180, 7))]
    ref = [make(capi, wl, precision, 3, 5) for wl in wls]
    got = [make(capi, wl, precision) for wl in wls]
    for n in (12, 1, 120):
        for s in ref:
            s.step_n(n)
        capi.step_many(got, n)
        for a, b in zip(ref, got):
            assert np.array_equal(a.read_populations(), b.read_populations()), n
    for s in ref + got:
        s.close()


def brick(N, shape, seed):
    """3-D as field()."""
    from inputs import components as C, fields as Fi
    if N <= 2:
        return W.random_droplet(N, shape, seed=seed, lattice=1)
    st = W.states()["spinodal10"]
    rho = Fi.add_noise(Fi.uniform(shape[0], shape[1], st["rho_uniform"][:N], nz=shape[2]), 1e-2,
                       seed)
    return W.Workload(C.N_ALKANES[:N], 325.0, rho, shape, kij=np.array(st["kij"])[:N, :N],
                      lattice=1)


def make3(capi, wl, precision):
    mix = wl.gpu_mixture()
    s = capi.Simulation(mix, 1, precision, wl.shape, wl.rho)
    s._mix = mix
    return s


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("N,shape,seed", [
    (2, (9, 8, 7), 21), (1, (70, 6, 5), 5), (2, (1, 5, 3), 21), (1, (5, 1, 1), 5),
    (2, (48, 33, 17), 21), (1, (61, 99, 97), 5), (2, (140, 73, 60), 21), (10, (85, 85, 71), 24), (7, (125, 45, 120), 4)])
def test_field_form_3d_matches_single_steps_bitwise(N, shape, seed, precision):
    """Runs on D3Q19 grids that take the field form (one and two components,
    and grids that fill the GPU; widths, heights and depths that leave ragged
    tiles, grids smaller than a tile's rim) against the same steps taken one at
    a time, which the multi-pass kernels do.  (The one-component drop is not
    an equilibrium and leaves the EOS domain during the last run: the same
    sites do so, with the same status.)"""
    capi = _capi()
    wl = brick(N, shape, seed)
    a, b = make3(capi, wl, precision), make3(capi, wl, precision)
    for n in (2, 1, 5, 67):
        for _ in range(n):
            a.step_n(1)
        b.step_n(n)
        assert np.array_equal(a.read_populations(), b.read_populations(), equal_nan=True), n
    assert a.diagnostics()["status"] == b.diagnostics()["status"]
    a.close()
    b.close()


def test_field_form_3d_batch_bitwise():
    """A batch whose members each take the field form, and one with a member
    too small for it."""
    capi = _capi()
    for shapes in (((70, 80, 75), (128, 64, 80)), ((70, 80, 75), (20, 11, 9))):
        wls = [brick(2, s, 21) for s in shapes]
        ref, got = [make3(capi, wl, 0) for wl in wls], [make3(capi, wl, 0) for wl in wls]
        for n in (3, 1, 40):
            for s in ref:
                for _ in range(n):
                    s.step_n(1)
            capi.step_many(got, n)
            for a, b in zip(ref, got):
                assert np.array_equal(a.read_populations(), b.read_populations()), (shapes, n)
        for s in ref + got:
            s.close()
