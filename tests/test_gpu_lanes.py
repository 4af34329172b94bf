"""Groups of a batch (component counts, precisions, lattices) stepped beside
each other on side streams: bitwise the simulations stepped alone, through run
lengths that take the side streams and ones that do not, on the null stream
and on streams that change from call to call with no host synchronisation,
with other work of a member (read-out, a run alone) between the calls.
"""
import numpy as np
import pytest

from tests import workloads as W
from tests.test_gpu_parity import _capi

pytestmark = pytest.mark.gpu

# component count, shape, seed, lattice, precision; draws that stay in the EOS
# domain over the steps taken
GROUPS = [(3, (67, 45), 31, 0, 0), (3, (130, 19), 31, 0, 1), (2, (200, 9), 31, 0, 1),
          (3, (61, 23), 52, 0, 0), (2, (48, 40, 36), 72, 1, 0), (2, (9, 8, 7), 5, 1, 1)]


def make(capi, spec):
    N, shape, seed, lattice, prec = spec
    wl = W.random_droplet(N, shape, seed=seed, lattice=lattice)
    mix = wl.gpu_mixture()
    s = capi.Simulation(mix, lattice, prec, shape, wl.rho)
    s._mix = mix
    return s


@pytest.mark.parametrize("members", [2, 4, 6])
def test_groups_beside_each_other_bitwise(members):
    import torch
    capi = _capi()
    specs = GROUPS[-members:]
    streams = [None, torch.cuda.Stream(), torch.cuda.Stream()]
    plan = [(0, 1), (1, 12), (2, 3), (1, 65), (0, 7), (2, 40)]
    sims = [make(capi, s) for s in specs]
    torch.cuda.synchronize()
    for k, n in plan:
        capi.step_many(sims, n, streams[k])
        if n == 3:
            sims[0].step_n(2, streams[1])     # a run alone, on another stream
            sims[-1].read_populations()
    for i, (spec, s) in enumerate(zip(specs, sims)):
        ref = make(capi, spec)
        ref.step_n(sum(n for _, n in plan) + (2 if i == 0 else 0))
        a, b = ref.read_populations(), s.read_populations()
        assert np.isfinite(a).all()
        assert np.array_equal(a, b), spec
        assert s.diagnostics()["step"] == ref.diagnostics()["step"]
        ref.close()
    for s in sims:
        s.close()
