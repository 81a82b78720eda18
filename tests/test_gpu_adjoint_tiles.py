"""GPU: the tile adjoint of column geometries (gjp_adjoint_tiles.hip) against the
FP64 oracle where it can go wrong: every candidate list (ray spacings along
axis 2 from a quarter of a voxel to several), tiles cut off on every axis, one
and two voxels per lane, detectors that leave the volume uncovered or reach
past it, reversed and slanted detector axes, and sources at the edge of the
rule that selects it. The bound is the stated one of an FP32 adjoint, relative
L2 1e-5 and every element within 1e-5 of the largest."""
import numpy as np
import pytest

from gpu_helpers import assert_parity, cuda, note

pytestmark = pytest.mark.gpu

TOL32 = 1e-5


@pytest.fixture(scope="module")
def gjp():
    import paper_1609_00958_amd as m
    return m


def _check(gjp, oracle_mod, G, seed, what):
    import torch
    og = oracle_mod.Geometry(G.shape, G.views, G.n_u, G.n_v,
                             beam=oracle_mod.CONE if G.beam == 0 else oracle_mod.PARALLEL,
                             voxel_size=G.voxel_size, center=G.center, weight=G.weight,
                             clip_cylinder=G.clip_cylinder)
    y = np.random.default_rng(seed).uniform(0, 1, size=G.sino_shape).astype(np.float32)
    note(f"tile adjoint {what}")
    x = gjp.back(torch.from_numpy(y).to(cuda()), G).cpu().numpy()
    assert_parity(x, oracle_mod.adjoint(og, y), TOL32)


@pytest.mark.parametrize("weight", ["linear", "spline"])
@pytest.mark.parametrize("pitch_v", [0.3, 0.6, 0.72, 0.9, 1.05, 1.3, 1.6, 2.2, 4.0])
def test_ray_spacings(gjp, oracle_mod, pitch_v, weight):
    n2 = 70 if weight == "linear" else 60  # two voxels per lane, one
    n_v = max(8, int(1.6 * n2 / pitch_v))
    G = gjp.Geometry.circular_cone((22, 26, n2), 7, 40, n_v, 120.0, 180.0, 1.1, pitch_v,
                                   weight=weight)
    _check(gjp, oracle_mod, G, 11, f"pitch_v {pitch_v} {weight}")


@pytest.mark.parametrize("beam", ["cone", "parallel"])
@pytest.mark.parametrize("shape,n_u,n_v", [((8, 8, 64), 12, 64), ((9, 17, 65), 31, 20),
                                           ((7, 23, 129), 9, 150), ((33, 5, 128), 60, 301),
                                           ((1, 40, 3), 50, 5), ((40, 1, 200), 3, 64)])
def test_ragged_sizes(gjp, oracle_mod, beam, shape, n_u, n_v):
    if beam == "cone":
        G = gjp.Geometry.circular_cone(shape, 13, n_u, n_v, 150.0, 260.0, 1.2, 1.3)
    else:
        G = gjp.Geometry.parallel(shape, 13, n_u, n_v, 0.8, 0.75)
    _check(gjp, oracle_mod, G, 12, f"{beam} {shape} {n_u}x{n_v}")


@pytest.mark.parametrize("case", ["flipped", "slanted", "anisotropic", "clipped", "shifted"])
@pytest.mark.parametrize("beam", ["cone", "parallel"])
def test_geometries(gjp, oracle_mod, beam, case):
    shape, n_views, n_u, n_v = (30, 21, 75), 70, 44, 90
    vs, ctr = (1.0, 1.0, 1.0), (0.0, 0.0, 0.0)
    if beam == "cone":
        v = gjp.views_circular_cone(n_views, 140.0, 220.0, 1.3, 1.25, n_u, n_v)
    else:
        v = gjp.views_parallel(n_views, 0.9, 0.85, n_u, n_v)
    if case == "flipped":
        v[:, 3:6] += (n_v - 1) * v[:, 9:12]
        v[:, 9:12] *= -1.0
    elif case == "slanted":
        v[:, 8] += 0.31          # du climbs along axis 2
        v[:, 5] -= 0.31 * 0.5 * (n_u - 1)
        v[:, 2] += 20.0 if beam == "cone" else 0.2
    elif case == "anisotropic":
        vs, ctr = (0.8, 1.25, 1.1), (2.0, -1.5, 3.0)
    elif case == "shifted":
        v[:, 3:6] += 9.3 * v[:, 6:9] - 21.7 * v[:, 9:12]  # off-centre detector
    G = gjp.Geometry(shape, v, n_u, n_v, beam=beam, voxel_size=vs, center=ctr,
                     clip_cylinder=case == "clipped")
    _check(gjp, oracle_mod, G, 13, f"{beam} {case}")


@pytest.mark.parametrize("sod", [30.0, 38.0, 45.0, 60.0])
def test_near_sources(gjp, oracle_mod, sod):
    """Wide fans whose views have columns of both driving axes; the nearest
    sources lie inside the rule's margin and take the gather instead."""
    G = gjp.Geometry.circular_cone((30, 34, 40), 24, 90, 60, sod, sod + 40.0, 1.4, 1.4)
    _check(gjp, oracle_mod, G, 14, f"source at {sod}")


@pytest.mark.parametrize("climb", [0.5, 6.0, 10.0, -10.0])
def test_columns_that_climb(gjp, oracle_mod, climb):
    """Neighbouring columns many rows apart along axis 2, rays a fiftieth of a voxel apart:
    up to more detector rows per tile than its window holds (those take the gather)."""
    shape, n_u, n_v = (24, 22, 60), 40, 3000
    v = gjp.views_parallel(5, 1.0, 0.02, n_u, n_v)[1:3].copy()
    v[:, 8] = climb
    v[:, 5] -= climb * 0.5 * (n_u - 1)
    G = gjp.Geometry(shape, v, n_u, n_v, beam="parallel")
    _check(gjp, oracle_mod, G, 15, f"columns climbing {climb}")


@pytest.mark.parametrize("n_views", [1, 3, 14])
@pytest.mark.parametrize("beam", ["cone", "parallel"])
@pytest.mark.parametrize("centre", [0, 45, 90, 170])
def test_views_of_one_axis(gjp, oracle_mod, beam, centre, n_views):
    """Views within a few degrees: columns of one driving axis (one pass over the volume, or
    partial volumes of that axis only) or, about 45 degrees, of both."""
    shape, n_u, n_v = (33, 30, 70), 50, 80
    v = (gjp.views_circular_cone(360, 200.0, 300.0, 1.2, 1.5, n_u, n_v) if beam == "cone"
         else gjp.views_parallel(360, 1.0, 0.9, n_u, n_v))
    v = v[[(centre + k - n_views // 2) % 360 for k in range(n_views)]]
    G = gjp.Geometry(shape, v, n_u, n_v, beam=beam)
    _check(gjp, oracle_mod, G, 18, f"{beam}, {n_views} views about {centre} degrees")


@pytest.mark.parametrize("views", [[0], [45], [10, 100]])
def test_few_views_of_a_large_volume(gjp, oracle_mod, views):
    """One pass, two of which the second adds to half of the tiles, two."""
    shape, n_u, n_v = (208, 204, 200), 90, 70
    v = gjp.views_circular_cone(360, 800.0, 1200.0, 5.0, 4.5, n_u, n_v)[views]
    _check(gjp, oracle_mod, gjp.Geometry(shape, v, n_u, n_v), 19, f"large volume, views {views}")
