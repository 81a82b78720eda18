"""GPU: the forward of general geometries against the FP64 oracle where the dealing of
its tiles to the XCDs and its groups of four planes can go wrong: fewer and more than
eight columns of tiles, ragged ends, one view and several, rays of one to five samples
on every driving axis. The bound is the stated one of an FP32 forward, relative L2
1e-5 and every element within 1e-5 of the largest. Batched calls (another launch
order) are bitwise equal."""
import numpy as np
import pytest

import workloads
from gpu_helpers import assert_parity, cuda, note

pytestmark = pytest.mark.gpu

TOL32 = 1e-5


@pytest.mark.parametrize("beam", ["cone", "parallel"])
@pytest.mark.parametrize("shape,n_views,n_u,n_v", [((20, 18, 22), 1, 5, 3), ((21, 17, 19), 9, 112, 17),
                                                   ((15, 24, 18), 4, 113, 40), ((16, 16, 16), 11, 150, 5),
                                                   ((5, 3, 4), 7, 33, 129), ((1, 2, 3), 12, 20, 20)])
def test_tiles(oracle_mod, beam, shape, n_views, n_u, n_v):
    import torch

    import paper_1609_00958_amd as gjp
    make = workloads.random_cone_views if beam == "cone" else workloads.random_parallel_views
    G = gjp.Geometry(shape, make(41, n_views, shape, n_u, n_v), n_u, n_v, beam=beam)
    og = oracle_mod.Geometry(G.shape, G.views, n_u, n_v,
                             beam=oracle_mod.CONE if beam == "cone" else oracle_mod.PARALLEL)
    x = np.random.default_rng(42).uniform(0, 1, size=shape).astype(np.float32)
    note(f"general forward {beam} {shape} {n_views} x {n_u} x {n_v}")
    d = torch.from_numpy(x).to(cuda())
    y = gjp.forward(d, G)
    assert_parity(y.cpu().numpy(), oracle_mod.forward(og, x), TOL32)
    assert torch.equal(gjp.forward_batched([d], [G])[0], y)


@pytest.mark.parametrize("n_u,n_v,n_views", [(1, 70, 3), (3, 200, 5), (4, 64, 9), (5, 130, 2), (8, 33, 4),
                                             (12, 90, 3), (40, 1, 30), (40, 2, 3), (300, 3, 30),
                                             (60, 15, 5)])
@pytest.mark.parametrize("beam", ["cone", "parallel"])
def test_narrow_detectors(oracle_mod, beam, n_u, n_v, n_views):
    """Few columns or rows: dealt tiles of every shape, and groups of views."""
    import torch

    import paper_1609_00958_amd as gjp
    shape = (19, 24, 17)
    make = workloads.random_cone_views if beam == "cone" else workloads.random_parallel_views
    G = gjp.Geometry(shape, make(43, n_views, shape, n_u, n_v), n_u, n_v, beam=beam)
    og = oracle_mod.Geometry(G.shape, G.views, n_u, n_v,
                             beam=oracle_mod.CONE if beam == "cone" else oracle_mod.PARALLEL)
    x = np.random.default_rng(44).uniform(0, 1, size=shape).astype(np.float32)
    note(f"general forward {beam} {n_views} x {n_u} x {n_v}")
    d = torch.from_numpy(x).to(cuda())
    y = gjp.forward(d, G)
    assert_parity(y.cpu().numpy(), oracle_mod.forward(og, x), TOL32)
    assert torch.equal(gjp.forward_batched([d], [G])[0], y)


@pytest.mark.parametrize("kind", ["column scan", "wide cone", "general"])
@pytest.mark.parametrize("dtype", ["float32", "float16"])
def test_autotuned_choice(oracle_mod, tmp_path, monkeypatch, kind, dtype):
    """Whichever kernels the autotuner chooses: the forward within the bound, batches
    bitwise equal to single calls, and the choice read back from the file."""
    import torch

    import paper_1609_00958_amd as gjp
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("GJP_TUNE_CACHE", str(path))
    shape, n_u, n_v = (24, 22, 30), 33, 30
    if kind == "general":
        G = gjp.Geometry(shape, workloads.random_cone_views(45, 7, shape, n_u, n_v), n_u, n_v)
    else:
        sod = 300.0 if kind == "column scan" else 26.0
        G = gjp.Geometry.circular_cone(shape, 7, n_u, n_v, sod, sod + 20.0, 1.1, 1.7)
    og = oracle_mod.Geometry(G.shape, G.views, n_u, n_v, beam=oracle_mod.CONE)
    x = torch.from_numpy(np.random.default_rng(46).uniform(0, 1, size=shape).astype(np.float32))
    x = x.to(getattr(torch, dtype))
    note(f"autotuned {kind} {dtype}")
    d = x.to(cuda())
    gjp.autotune(d, G)
    y = gjp.forward(d, G)
    assert_parity(y.cpu().numpy(), oracle_mod.forward(og, x.float().numpy()), TOL32)
    assert torch.equal(gjp.forward_batched([d], [G])[0], y)
    gjp.reset_forward_tile(G, getattr(torch, dtype))  # the file's entry applies
    assert torch.equal(gjp.forward(d, G), y)
    for entry in path.read_text().splitlines():
        assert len(entry.split()) in (5, 6)


@pytest.mark.parametrize("tile", [192, 64, 16])
def test_batched_views_in_columns(oracle_mod, tile):
    """General geometry with a few views whose columns lie along axis 2: single calls
    take the rule's kernel whatever tile is set, batched ones give the same bits."""
    import torch

    import paper_1609_00958_amd as gjp
    shape, n_u, n_v = (40, 36, 50), 64, 400
    views = gjp.views_circular_cone(9, 160.0, 320.0, 1.0, 0.3, n_u, n_v).reshape(9, 12)
    views[2:, 9] = 0.01  # seven of nine tilted
    G = gjp.Geometry(shape, views, n_u, n_v)
    og = oracle_mod.Geometry(G.shape, G.views, n_u, n_v, beam=oracle_mod.CONE)
    x = np.random.default_rng(47).uniform(0, 1, size=shape).astype(np.float32)
    note(f"general forward with columns, tile {tile}")
    d = torch.from_numpy(x).to(cuda())
    gjp.set_forward_tile(G, torch.float32, tile, 8, 4)
    try:
        y = gjp.forward(d, G)
        assert_parity(y.cpu().numpy(), oracle_mod.forward(og, x), TOL32)
        assert torch.equal(gjp.forward_batched([d], [G])[0], y)
    finally:
        gjp.reset_forward_tile(G, torch.float32)
