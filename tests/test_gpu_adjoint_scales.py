"""Scales of large planes, which several workgroups look for: the largest part of 2 dL/dI E in the first,
a middle and the last run of the pixels (a scale that missed it would leave the range of the halves)."""
import numpy as np
import pytest

from tests.helpers import rel_l2
from tests.test_gpu_adjoint_tiles import TOL, _run

pytestmark = pytest.mark.gpu


# runs of 4096 pixels or more: one, two, three runs of unequal length, and one plane of many
@pytest.mark.parametrize("nx,ny,nz,n_stacks", [(64, 112, 2, 1), (80, 112, 3, 2), (112, 112, 2, 1), (272, 256, 1, 1)])
@pytest.mark.parametrize("at", [0, 1, 2])
def test_largest_part_anywhere(lib, nx, ny, nz, n_stacks, at):
    def gradient(I):
        g = I - 0.3 * I.max()
        g[0, 0].flat[(0, nx * ny // 2 + 3, nx * ny - 1)[at]] = 1e9 * I.max() / I[0, 0].min()
        return g

    here, (dc_ref, dw_ref) = _run(lib, 64, nx, ny, nz, n_stacks, gradient)
    dc, dw = here()
    assert rel_l2(dc, dc_ref) < TOL
    assert rel_l2(dw, dw_ref) < TOL
