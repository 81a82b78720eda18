"""GPU: adjoints whose scratch holds part of the views at a time (scaled rays of 2 GiB,
ray tables of 512 MiB): the later chunks add to the volume, the last one is shorter and
splits its views differently. A call over all views against the sum of calls over a few
views each, which are single chunks (those are compared with the oracle elsewhere). Both
are FP32 adjoints within the stated relative L2 of 1e-5 and 1e-5 of the largest value."""
import numpy as np
import pytest

from gpu_helpers import assert_parity, cuda, note

pytestmark = pytest.mark.gpu

TOL32 = 1e-5


def _check(shape, views, n_u, n_v, beam, parts, what):
    import torch

    import paper_1609_00958_amd as gjp
    dev = cuda()
    g = torch.Generator(dev).manual_seed(61)
    y = torch.empty((len(views), n_u, n_v), device=dev).uniform_(0.5, 1.0, generator=g)
    note(f"adjoint in chunks: {what}")
    x = gjp.back(y, gjp.Geometry(shape, views, n_u, n_v, beam=beam)).double()
    want = torch.zeros(shape, dtype=torch.float64, device=dev)
    for k in range(0, len(views), parts):
        note(f"views from {k}")
        G = gjp.Geometry(shape, views[k:k + parts], n_u, n_v, beam=beam)
        want += gjp.back(y[k:k + parts].contiguous(), G).double()
    assert_parity(x.cpu().numpy(), want.cpu().numpy(), TOL32)


def test_tiles_with_partial_volumes():
    """64 MiB of rays per view: 32 views, then 8."""
    import paper_1609_00958_amd as gjp
    v = gjp.views_circular_cone(40, 256.0, 512.0, 0.05, 0.15, 4096, 4096)
    _check((64, 64, 64), v, 4096, 4096, "cone", 10, "64^3, 40 views of 4096^2")


def test_tiles_into_the_volume():
    """32 MiB of rays per view, a volume too large for partial ones: 64 views, then 3."""
    import paper_1609_00958_amd as gjp
    v = gjp.views_circular_cone(67, 1400.0, 2100.0, 0.25, 0.4, 4096, 2048)
    _check((340, 328, 336), v, 4096, 2048, "cone", 30, "336^3, 67 views of 4096 x 2048")


def test_cube_gather():
    """32 MB of rays per view: 16 views, then 5."""
    rng = np.random.default_rng(62)
    shape, n, views = (40, 36, 33), 1000, []
    for _ in range(21):
        w, t = rng.normal(size=(2, 3))
        w /= np.linalg.norm(w)
        e1 = t - w * (t @ w)
        e1 /= np.linalg.norm(e1)
        du, dv = 0.1 * e1, 0.1 * np.cross(w, e1)
        views.append(np.concatenate([-w, -0.5 * (n - 1) * (du + dv), du, dv]))
    _check(shape, np.array(views), n, n, "parallel", 7, "general 40 x 36 x 33, 21 views of 1000^2")
