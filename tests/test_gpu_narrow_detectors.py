"""GPU: adjoints of general geometries whose detectors are narrower than the image of a
few voxels, against the FP64 oracle: one to sixteen rows or columns at pitches from a
tenth of a voxel to one, circular about axes 0 and 1 and oblique, cone and parallel, and
sources so near that a cube's image is wider than an ordinary detector. The bound is the
stated one of an FP32 adjoint, relative L2 1e-5 and every element within 1e-5 of the
largest."""
import numpy as np
import pytest

from gpu_helpers import assert_parity, cuda, note

pytestmark = pytest.mark.gpu

TOL32 = 1e-5


def _about(axis, v):
    """Views circular about axis 2, turned to another axis."""
    order = {0: [2, 0, 1], 1: [0, 2, 1]}[axis]
    return np.ascontiguousarray(v.reshape(-1, 4, 3)[:, :, order].reshape(-1, 12))


def _oblique(beam, n_views, n_u, n_v, pitch, sod, sdd):
    rng = np.random.default_rng(51)
    out = []
    for _ in range(n_views):
        w, t = rng.normal(size=(2, 3))
        w /= np.linalg.norm(w)
        e1 = t - w * (t @ w)
        e1 /= np.linalg.norm(e1)
        e2 = np.cross(w, e1)
        mid = (sod - sdd) * w if beam == "cone" else np.zeros(3)
        du, dv = pitch * e1, pitch * e2
        out.append(np.concatenate([sod * w if beam == "cone" else -w,
                                   mid - 0.5 * (n_u - 1) * du - 0.5 * (n_v - 1) * dv, du, dv]))
    return np.array(out)


def _check(oracle_mod, shape, views, n_u, n_v, beam, what):
    import torch

    import paper_1609_00958_amd as gjp
    G = gjp.Geometry(shape, views, n_u, n_v, beam=beam)
    og = oracle_mod.Geometry(shape, views, n_u, n_v,
                             beam=oracle_mod.CONE if beam == "cone" else oracle_mod.PARALLEL)
    y = np.random.default_rng(52).uniform(0.5, 1, size=G.sino_shape).astype(np.float32)
    note(f"narrow detector {what} {beam} {shape} {n_u}x{n_v}")
    want = oracle_mod.adjoint(og, y)
    assert (want != 0).any()
    assert_parity(gjp.back(torch.from_numpy(y).to(cuda()), G).cpu().numpy(), want, TOL32)


@pytest.mark.parametrize("swap", [False, True])
@pytest.mark.parametrize("narrow,pitch", [(1, 1.0), (1, 0.5), (2, 1.0), (3, 0.3), (4, 0.25),
                                          (8, 0.25), (16, 0.1)])
@pytest.mark.parametrize("beam", ["cone", "parallel"])
@pytest.mark.parametrize("scan", ["axis 0", "axis 1", "oblique"])
def test_narrow(oracle_mod, scan, beam, narrow, pitch, swap):
    import paper_1609_00958_amd as gjp
    n_u, n_v = (narrow, 37) if swap else (37, narrow)
    shape = {"axis 0": (5, 24, 21), "axis 1": (24, 5, 21), "oblique": (24, 20, 21)}[scan]
    if scan == "oblique":
        views = _oblique(beam, 3, n_u, n_v, pitch, 60.0, 90.0)
    else:
        views = (gjp.views_circular_cone(3, 60.0, 90.0, pitch, pitch, n_u, n_v) if beam == "cone"
                 else gjp.views_parallel(3, pitch, pitch, n_u, n_v))
        views = _about(int(scan[-1]), views)
    _check(oracle_mod, shape, views, n_u, n_v, beam, f"{scan} pitch {pitch}")


@pytest.mark.parametrize("n", [1, 5, 40])
def test_near_source(oracle_mod, n):
    """A source three to twenty voxels from the grid: images of a cube from a few pixels
    to the whole detector."""
    shape = (20, 22, 18)
    _check(oracle_mod, shape, _oblique("cone", 6, n, n, 40.0 / n, 19.0, 60.0), n, n, "cone", "near")
