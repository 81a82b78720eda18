"""GPU: the gather adjoint of general geometries (gjp_adjoint_free.hip) against the
FP64 oracle where it can go wrong: tiles cut off on every axis, all three driving
axes, rays from many per voxel (a tile's rectangle staged in parts) to fewer than
one, detectors that leave the volume uncovered or reach past it, sources near the
grid (inside the rule's margin the tile splat takes over), views split over
workgroups, and values that are not finite. The bound is the stated one of an FP32
adjoint, relative L2 1e-5 and every element within 1e-5 of the largest."""
import numpy as np
import pytest

import workloads
from gpu_helpers import assert_parity, cuda, note

pytestmark = pytest.mark.gpu

TOL32 = 1e-5


@pytest.fixture(scope="module")
def gjp():
    import paper_1609_00958_amd as m
    return m


def _oracle(oracle_mod, G):
    return oracle_mod.Geometry(G.shape, G.views, G.n_u, G.n_v,
                               beam=oracle_mod.CONE if G.beam == 0 else oracle_mod.PARALLEL,
                               voxel_size=G.voxel_size, center=G.center, weight=G.weight,
                               clip_cylinder=G.clip_cylinder)


def _check(gjp, oracle_mod, G, seed, what):
    import torch
    y = np.random.default_rng(seed).uniform(0, 1, size=G.sino_shape).astype(np.float32)
    note(f"free adjoint {what}")
    x = gjp.back(torch.from_numpy(y).to(cuda()), G).cpu().numpy()
    assert_parity(x, oracle_mod.adjoint(_oracle(oracle_mod, G), y), TOL32)


def _views(beam, seed, n_views, shape, n_u, n_v):
    make = workloads.random_cone_views if beam == "cone" else workloads.random_parallel_views
    return make(seed, n_views, shape, n_u, n_v)


@pytest.mark.parametrize("weight", ["linear", "spline"])
@pytest.mark.parametrize("beam", ["cone", "parallel"])
@pytest.mark.parametrize("shape,n_views,n_u,n_v", [((16, 16, 8), 5, 20, 20), ((17, 33, 9), 9, 40, 31),
                                                   ((30, 15, 41), 40, 64, 50), ((3, 40, 2), 6, 50, 12),
                                                   ((24, 20, 28), 4, 3, 70), ((20, 22, 18), 5, 150, 170)])
def test_sizes(gjp, oracle_mod, beam, shape, n_views, n_u, n_v, weight):
    G = gjp.Geometry(shape, _views(beam, 31, n_views, shape, n_u, n_v), n_u, n_v, beam=beam,
                     weight=weight)
    _check(gjp, oracle_mod, G, 32, f"{beam} {shape} {n_u}x{n_v} {weight}")


@pytest.mark.parametrize("pitch", [0.2, 0.5, 3.0])
@pytest.mark.parametrize("beam", ["cone", "parallel"])
def test_pitches(gjp, oracle_mod, beam, pitch):
    shape, n_u, n_v = (14, 18, 13), 90, 80
    v = _views(beam, 33, 6, shape, n_u, n_v)
    # the same detectors' centres with another pitch
    mid = v[:, 3:6] + 0.5 * (n_u - 1) * v[:, 6:9] + 0.5 * (n_v - 1) * v[:, 9:12]
    v[:, 6:12] *= pitch
    v[:, 3:6] = mid - 0.5 * (n_u - 1) * v[:, 6:9] - 0.5 * (n_v - 1) * v[:, 9:12]
    G = gjp.Geometry(shape, v, n_u, n_v, beam=beam, voxel_size=(0.9, 1.2, 1.1),
                     center=(1.0, -2.0, 0.5))
    _check(gjp, oracle_mod, G, 34, f"{beam} pitch x {pitch}")


@pytest.mark.parametrize("clip", [False, True])
@pytest.mark.parametrize("scale", [0.35, 0.5, 0.7])
def test_near_sources(gjp, oracle_mod, scale, clip):
    shape, n_u, n_v = (22, 20, 24), 40, 44
    v = _views("cone", 35, 8, shape, n_u, n_v)
    v[:, 0:3] *= scale
    G = gjp.Geometry(shape, v, n_u, n_v, beam="cone", clip_cylinder=clip)
    _check(gjp, oracle_mod, G, 36, f"sources x {scale}, clip {clip}")


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_non_finite_rays_reach_their_voxels_only(gjp, oracle_mod, bad):
    import torch
    shape, n_views, n_u, n_v = (18, 20, 16), 4, 24, 26
    G = gjp.Geometry(shape, _views("cone", 37, n_views, shape, n_u, n_v), n_u, n_v, beam="cone")
    og = _oracle(oracle_mod, G)
    y = np.random.default_rng(38).uniform(0.5, 1, size=G.sino_shape).astype(np.float32)
    clean = oracle_mod.adjoint(og, y)
    hit = np.zeros(G.sino_shape, np.float32)
    hit[1, n_u // 2, n_v // 2] = 1.0
    weight = oracle_mod.adjoint(og, hit)
    y[1, n_u // 2, n_v // 2] = bad
    note(f"free adjoint, {bad} ray")
    x = gjp.back(torch.from_numpy(y).to(cuda()), G).cpu().numpy()
    assert (weight > 1e-3).any() and not np.isfinite(x[weight > 1e-3]).any()
    far = weight == 0.0
    assert np.isfinite(x[far]).all()
    assert_parity(x[far], clean[far], TOL32)
