"""GPU: the row forward of column geometries (gjp_forward_rows.hip) against the
FP64 oracle where it can go wrong: two, three, four and six rays per lane, windows
of one load, one and a tail, and two, rows cut off inside a load of four voxels,
detectors that reach past the volume on either side, reversed and slanted axes,
every storage type (16-bit rows of odd length take the padded copies), and batches
bitwise equal to single calls. The bound is the stated one of an FP32 forward,
relative L2 1e-5 and every element within 1e-5 of the largest; 16-bit volumes are
compared with the oracle on the rounded volume, so theirs is the same."""
import numpy as np
import pytest

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


def _check(gjp, oracle_mod, G, seed, what, dtype="float32"):
    import torch
    x = torch.from_numpy(np.random.default_rng(seed).uniform(0, 1, size=G.shape)
                         .astype(np.float32)).to(getattr(torch, dtype))
    note(f"row forward {what} {dtype}")
    y = gjp.forward(x.to(cuda()), G).cpu().numpy()
    assert_parity(y, oracle_mod.forward(_oracle(oracle_mod, G), x.float().numpy()), TOL32)


# rays per lane by the detector's length; windows by the ray spacing
@pytest.mark.parametrize("weight", ["linear", "spline"])
@pytest.mark.parametrize("n2", [1, 40, 254, 255, 330])
@pytest.mark.parametrize("n_v,pitch_v", [(5, 1.5), (128, 0.5), (130, 1.5), (192, 2.0), (193, 1.2),
                                         (256, 1.6), (257, 2.4), (384, 1.0), (384, 1.15),
                                         (400, 1.8), (100, 4.5), (150, 9.0)])
def test_windows(gjp, oracle_mod, n_v, pitch_v, n2, weight):
    G = gjp.Geometry.circular_cone((9, 12, n2), 3, 11, n_v, 400.0, 600.0, 1.5, pitch_v,
                                   weight=weight)
    _check(gjp, oracle_mod, G, 21, f"{n_v} rays, pitch {pitch_v}, n2 {n2}, {weight}")


@pytest.mark.parametrize("dtype", ["float32", "bfloat16", "float16"])
@pytest.mark.parametrize("beam", ["cone", "parallel"])
@pytest.mark.parametrize("shape,n_u,n_v", [((8, 8, 64), 12, 64), ((9, 17, 66), 31, 200),
                                           ((7, 131, 258), 9, 301), ((70, 5, 127), 30, 150),
                                           ((1, 40, 2), 50, 5), ((40, 1, 200), 3, 130)])
def test_ragged_sizes(gjp, oracle_mod, beam, shape, n_u, n_v, dtype):
    if beam == "cone":
        G = gjp.Geometry.circular_cone(shape, 6, n_u, n_v, 250.0, 360.0, 1.2, 1.3)
    else:
        G = gjp.Geometry.parallel(shape, 6, n_u, n_v, 0.8, 0.75)
    _check(gjp, oracle_mod, G, 22, f"{beam} {shape} {n_u}x{n_v}", dtype)


@pytest.mark.parametrize("case", ["flipped", "slanted", "anisotropic", "clipped", "shifted"])
@pytest.mark.parametrize("beam", ["cone", "parallel"])
def test_geometries(gjp, oracle_mod, beam, case):
    shape, n_views, n_u, n_v = (30, 21, 75), 17, 44, 210
    vs, ctr = (1.0, 1.0, 1.0), (0.0, 0.0, 0.0)
    if beam == "cone":
        v = gjp.views_circular_cone(n_views, 140.0, 220.0, 1.3, 0.9, n_u, n_v)
    else:
        v = gjp.views_parallel(n_views, 0.9, 0.6, n_u, n_v)
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
        v[:, 3:6] += 9.3 * v[:, 6:9] - 41.7 * v[:, 9:12]  # off-centre detector
    G = gjp.Geometry(shape, v, n_u, n_v, beam=beam, voxel_size=vs, center=ctr,
                     clip_cylinder=case == "clipped")
    _check(gjp, oracle_mod, G, 23, f"{beam} {case}")


@pytest.mark.parametrize("sod", [12.0, 20.0, 45.0])
def test_near_sources(gjp, oracle_mod, sod):
    """Sources inside and beside the grid: wide fans, steep climbs, and rays that
    the window's rule sends to the padded copies."""
    G = gjp.Geometry.circular_cone((30, 34, 40), 24, 90, 130, sod, sod + 40.0, 1.4, 0.7)
    _check(gjp, oracle_mod, G, 24, f"source at {sod}")


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("at", [(0, 0, 0), (11, 8, 39), (5, 3, 17), (0, 8, 39)])
def test_non_finite_voxels_reach_their_rays_only(gjp, oracle_mod, at, bad):
    import torch
    shape = (12, 9, 40)
    G = gjp.Geometry.circular_cone(shape, 12, 15, 140, 60.0, 90.0, 1.5, 0.6, clip_cylinder=False)
    og = _oracle(oracle_mod, G)
    x = np.random.default_rng(25).uniform(0.5, 1, size=shape).astype(np.float32)
    clean = oracle_mod.forward(og, x)
    hit = np.zeros(shape, np.float32)
    hit[at] = 1.0
    weight = oracle_mod.forward(og, hit)
    x[at] = bad
    note(f"row forward, {bad} at {at}")
    y = gjp.forward(torch.from_numpy(x).to(cuda()), G).cpu().numpy()
    assert not np.isfinite(y[weight > 1e-4]).any()
    # rays that pass within rounding of the voxel's reach may take it with weight 0
    near = np.zeros(shape, np.float32)
    near[tuple(slice(max(a - 1, 0), a + 2) for a in at)] = 1.0
    far = oracle_mod.forward(og, near) == 0.0
    assert far.any() and np.isfinite(y[far]).all()
    assert_parity(y[far], clean[far], TOL32)
    if np.isinf(bad):
        assert np.isposinf(y[weight > 1e-4]).all()


def test_batch_equals_single_calls(gjp):
    import torch
    dev = cuda()
    geoms, vols = [], []
    gen = torch.Generator().manual_seed(26)
    for k, (n2, n_v, pitch, dt) in enumerate([(64, 128, 0.9, torch.float32),
                                              (80, 192, 0.9, torch.float32),
                                              (75, 256, 0.6, torch.bfloat16),
                                              (75, 256, 0.6, torch.float32),
                                              (128, 384, 0.6, torch.float16),
                                              (127, 384, 0.6, torch.float16),
                                              (33, 150, 9.0, torch.float32)]):
        geoms.append(gjp.Geometry.circular_cone((20 + k, 31 - k, n2), 9, 21, n_v, 200.0, 300.0, 1.2,
                                                pitch, weight="spline" if k % 3 == 1 else "linear"))
        vols.append(torch.rand(geoms[-1].shape, generator=gen).to(dt).to(dev))
    # a 16-bit volume that starts on an odd element
    geoms.append(gjp.Geometry.circular_cone((20, 20, 64), 9, 21, 128, 200.0, 300.0, 1.2, 0.9))
    vols.append(torch.rand(20 * 20 * 64 + 1, generator=gen).half().to(dev)[1:].view(20, 20, 64))
    note("batched row forward")
    for _ in range(2):
        for y, g, x in zip(gjp.forward_batched(vols, geoms), geoms, vols):
            assert torch.equal(y, gjp.forward(x, g))


@pytest.mark.parametrize("z", [-178.5, -120.0, 178.5])
@pytest.mark.parametrize("pitch_v", [3.5, 3.55, 3.6])
def test_thin_volumes_seen_steeply(gjp, oracle_mod, pitch_v, z):
    """Four planes, rays that climb nearly a voxel per plane from far below or above:
    windows whose lower part lies beside the grid, at the limit of the rule."""
    shape, n_v = (4, 4, 240), 256
    v = gjp.views_circular_cone(2, 238.0, 476.0, 1.0, pitch_v, 3, n_v)[1:].copy()
    v[:, 2] = z
    G = gjp.Geometry(shape, v, 3, n_v, beam="cone")
    _check(gjp, oracle_mod, G, 27, f"thin volume, source at height {z}, pitch {pitch_v}")
