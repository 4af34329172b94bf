"""The fused D2Q9 step for items of one or two rows (all rows of an item at
once; variant 2 of set_tuning with rows <= 2) against the marching kernels:
bitwise the same populations, over component counts 1 ... 10, widths either
side of the 60-column strips, heights that leave a last item of one row,
grids narrower than a strip and lower than the halo, both precisions,
tau = 1 and 0.8, and the other cubics."""
import numpy as np
import pytest

from tests import workloads as W
from tests.test_gpu_field_form import field, make
from tests.test_gpu_parity import _capi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("N,shape,seed,tau,eos", [
    (1, (61, 23), 9, 1.0, "PR"), (2, (5, 5), 3, 1.0, "PR"), (2, (3, 70), 4, 0.8, "PR"),
    (3, (67, 45), 31, 0.8, "PR"), (3, (200, 2), 5, 1.0, "PR"), (4, (130, 75), 11, 1.0, "PR"),
    (5, (130, 1), 4, 1.0, "PR"), (6, (61, 29), 4, 0.8, "PR"), (7, (125, 17), 4, 1.0, "PR"),
    (8, (59, 8), 4, 1.0, "PR"), (9, (120, 7), 4, 1.0, "PR"), (10, (121, 19), 4, 0.8, "PR"),
    (3, (64, 9), 31, 1.0, "SRK"), (2, (62, 11), 11, 1.0, "vdW")])
def test_one_and_two_row_items_match_marching_bitwise(N, shape, seed, tau, eos, precision):
    capi = _capi()
    wl = W.random_droplet(N, shape, seed=seed, eos=eos) if N <= 4 else field(N, shape, seed)
    wl.tau = tau
    ref = make(capi, wl, precision, 3, 3)
    sims = [make(capi, wl, precision, 2, r) for r in (1, 2)]
    for n in (1, 2, 70):
        ref.step_n(n)
        g = ref.read_populations()
        for s in sims:
            s.step_n(n)
            assert np.array_equal(s.read_populations(), g), n
    assert np.all(np.isfinite(g))
    for s in sims + [ref]:
        s.close()
