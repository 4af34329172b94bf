"""Runs in a form fixed by fuglbm_set_form against runs that keep populations
at every step (kernels fixed by set_tuning): bitwise the same state, and the
form that was asked for is the one that ran.  Unlike the runs whose form the
trials choose, these reach every kernel at every size: all component counts,
the three cubics, heights down to one row, widths below a strip, rows per item
that leave remainders, run lengths below and above the graphs', batches, and a
stream that the caller captures."""
import numpy as np
import pytest

from tests import workloads as W
from tests.test_gpu_field_form import brick, field, make, make3
from tests.test_gpu_parity import _capi

pytestmark = pytest.mark.gpu

POPULATIONS, FIELDS, SINGLE = 1, 2, 3

# N, shape, seed, cubic, rows per item of the field form (0: the library's)
PLANES = [(1, (130, 75), 9, "PR", 0), (1, (61, 2), 9, "PR", 1), (2, (5, 5), 3, "PR", 2),
          (2, (62, 41), 11, "vdW", 0), (3, (67, 45), 31, "PR", 7), (3, (64, 37), 31, "SRK", 0),
          (3, (200, 3), 5, "PR", 3), (3, (3, 70), 31, "PR", 0), (4, (125, 33), 11, "PR", 10),
          (5, (121, 1), 4, "PR", 0), (5, (60, 58), 4, "PR", 29), (6, (59, 4), 4, "PR", 3),
          (7, (119, 31), 4, "PR", 0), (8, (61, 30), 4, "PR", 11), (9, (120, 7), 4, "PR", 4),
          (10, (1, 9), 4, "PR", 0), (10, (131, 26), 4, "PR", 0)]
CUBES = [(1, (9, 8, 7), 5, "PR"), (2, (30, 17, 15), 21, "SRK"), (2, (33, 15, 12), 21, "vdW"),
         (3, (17, 9, 5), 4, "PR"), (4, (70, 5, 3), 4, "PR"), (5, (12, 29, 11), 4, "PR"),
         (6, (29, 31, 1), 4, "PR"), (8, (1, 3, 40), 4, "PR"), (9, (61, 15, 9), 4, "PR"),
         (10, (28, 14, 26), 4, "PR")]
RUNS = (1, 2, 9, 3, 70)


def plane(N, shape, seed, eos):
    return (W.random_droplet(N, shape, seed=seed, eos=eos) if 1 < N <= 4 else
            field(N, shape, seed))


def cube(N, shape, seed, eos):
    return (W.random_droplet(N, shape, seed=seed, lattice=1, eos=eos) if N <= 2 else
            brick(N, shape, seed))


def fixed(s, form, rows=0):
    s.set_tuning(0, rows)
    s.set_form(form)
    return s


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("N,shape,seed,eos,rows", PLANES)
def test_planes_bitwise(N, shape, seed, eos, rows, precision):
    capi = _capi()
    wl = plane(N, shape, seed, eos)
    ref = make(capi, wl, precision, 2, 5)
    forms = [FIELDS, SINGLE] if N <= 3 else [FIELDS]
    sims = [fixed(make(capi, wl, precision), f, rows) for f in forms]
    for n in RUNS:
        ref.step_n(n)
        g = ref.read_populations()
        assert ref.form() == POPULATIONS
        for s, f in zip(sims, forms):
            s.step_n(n)
            assert s.form() == f
            assert np.array_equal(s.read_populations(), g), (n, f)
    assert np.all(np.isfinite(g))
    for s in sims + [ref]:
        assert s.diagnostics()["status"] == 0
        s.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("N,shape,seed,eos", CUBES)
def test_cubes_bitwise(N, shape, seed, eos, precision):
    capi = _capi()
    wl = cube(N, shape, seed, eos)
    ref, got = make3(capi, wl, precision), make3(capi, wl, precision)
    ref.set_tuning(1)
    got.set_form(FIELDS)
    for n in RUNS:
        ref.step_n(n)
        got.step_n(n)
        assert (ref.form(), got.form()) == (POPULATIONS, FIELDS)
        g = ref.read_populations()
        assert np.array_equal(got.read_populations(), g), n
    assert np.all(np.isfinite(g))
    for s in (ref, got):
        assert s.diagnostics()["status"] == 0
        s.close()


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("form", [FIELDS, SINGLE])
def test_batches_bitwise(form, precision):
    """One table of planes whose items end in remainders, from either buffer."""
    capi = _capi()
    wls = [plane(3, s, 31, "PR") for s in ((67, 45), (3, 70), (130, 19), (61, 23))]
    ref = [make(capi, wl, precision, 3, 5) for wl in wls]
    got = [fixed(make(capi, wl, precision), form) for wl in wls]
    got[1].set_form(POPULATIONS)
    got[1].step_n(1)                       # its state lies in the other buffer
    ref[1].step_n(1)
    got[1].set_form(form)
    for n in (2, 1, 70):
        for s in ref:
            s.step_n(n)
        capi.step_many(got, n)
        for a, b in zip(ref, got):
            assert b.form() == form
            assert np.array_equal(a.read_populations(), b.read_populations()), n
    for s in ref + got:
        s.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_members_of_other_forms_in_a_batch_bitwise(precision):
    """Groups that are split: planes at tau = 1 beside one at tau = 0.8 and one
    with fixed rows, and a large cube beside a small one and one whose form is
    fixed; every member ends where it ends alone."""
    capi = _capi()

    def sims():
        out = [make(capi, plane(3, s, 31, "PR"), precision) for s in ((301, 240), (256, 256), (61, 400))]
        wl = plane(3, (61, 23), 31, "PR")
        wl.tau = 0.8
        out.append(make(capi, wl, precision))
        out.append(make(capi, plane(3, (67, 45), 31, "PR"), precision, 2, 2))
        out += [make3(capi, cube(2, s, 21, "PR"), precision) for s in ((96, 96, 96), (8, 7, 9), (20, 11, 9))]
        out[-2].set_tuning(1)
        out[-1].set_form(FIELDS)
        return out

    ref, got = sims(), sims()
    for n in (12, 1, 70):
        for s in ref:
            s.step_n(n)
        capi.step_many(got, n)
        for k, (a, b) in enumerate(zip(ref, got)):
            assert np.array_equal(a.read_populations(), b.read_populations()), (n, k)
        forms = [s.form() for s in got]
        assert forms[3:5] == [POPULATIONS] * 2
        assert forms[5:] == [FIELDS if n > 1 else POPULATIONS, POPULATIONS, FIELDS]
    for s in ref + got:
        assert s.diagnostics()["status"] == 0
        s.close()


@pytest.mark.parametrize("N,shape,lattice", [(3, (67, 45), 0), (6, (59, 24), 0), (2, (30, 17, 15), 1)])
def test_captured_run_replayed(N, shape, lattice):
    """A run in field form on a stream that the caller captures: each replay,
    with read-outs of the library and other work on the device between them,
    is one more run."""
    import torch
    capi = _capi()
    wl = cube(N, shape, 21, "PR") if lattice else plane(N, shape, 31 if N == 3 else 4, "PR")
    ref, got = [(make3 if lattice else make)(capi, wl, 0) for _ in range(2)]
    ref.set_tuning(1 if lattice else 2, 0 if lattice else 5)
    got.set_form(FIELDS)
    st = torch.cuda.Stream()
    got.step_n(2, st)
    ref.step_n(2)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        got.step_n(7, st)
    assert got.form() == FIELDS
    torch.cuda.synchronize()
    a = torch.ones(1 << 20, device="cuda")
    for k in range(4):
        with torch.cuda.stream(st):
            graph.replay()
        ref.step_n(7)
        a.mul_(1.5).zero_()
        assert np.array_equal(got.read_populations(), ref.read_populations()), k
    for s in (ref, got):
        s.close()
