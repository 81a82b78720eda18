"""GPU: rays that leave the grid at its upper ends, one at a time, against the FP64
oracle: samples past the end are none of the forward's and have to weigh exactly
nothing in the adjoint, however small a weight would be (a SART update multiplies it by
the residual of a ray whose own sum is a sliver). On the samples the bound is 2^-22: a
weight's FP32 rounding (2^-24) and the step length's."""
import numpy as np
import pytest

from conftest import grid_point
from gpu_helpers import cuda, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [9, 10, 113])
@pytest.mark.parametrize("axis", [0, 1])
def test_samples_past_the_end_weigh_nothing(oracle_mod, axis, n):
    import torch

    import paper_1609_00958_amd as gjp
    shape = (40, n, 4) if axis == 0 else (n, 40, 4)
    slope = 0.011
    d, o, du = np.zeros(3), np.zeros(3), np.zeros(3)
    d[axis], d[1 - axis], du[1 - axis] = 1.0, slope, 1.0
    o[1 - axis] = n - 20.4 * slope  # out between planes 20 and 21
    v = np.concatenate([d, grid_point(shape, o), du, [0.0, 0.0, 1.0]])[None]
    G = gjp.Geometry(shape, v, 1, 4, beam="parallel")
    y = np.zeros(G.sino_shape, np.float32)
    y[0, 0, 1] = 1.0
    note(f"ray out of {shape} along axis {axis}")
    x = gjp.back(torch.from_numpy(y).to(cuda()), G).cpu().numpy()
    want = oracle_mod.adjoint(oracle_mod.Geometry(shape, v, 1, 4, beam=oracle_mod.PARALLEL), y)
    assert (want != 0).any()
    assert np.all(x[want == 0] == 0)
    assert np.abs(x - want).max() <= 2.0 ** -22
