"""The library's host rules on the CPU: which kernels a geometry is sent to, that every
geometry that a rule sends to a kernel has windows that fit that kernel's LDS arrays, and
what the adjoint does where the device has little room. csrc/gjp_api.cpp is compiled for
the host and driven by tests/host/planning_driver.cpp, over random geometries and the
ones at a rule's edge, with stand-ins for the launchers and the allocator."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "host")
CSRC = os.path.join(ROOT, "paper_1609_00958_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, " ".join(cmd) + "\n" + r.stdout[-3000:] + r.stderr[-3000:]
    return r.stdout


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    out = tmp_path_factory.mktemp("planning")
    objs = []
    for src in (os.path.join(CSRC, "gjp_api.cpp"), os.path.join(HERE, "planning_driver.cpp")):
        objs.append(str(out / (os.path.basename(src) + ".o")))
        _run([HIPCC, "-x", "hip", "--cuda-host-only", "-O2", "-std=c++17", "-ffp-contract=off",
              "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", src, "-o", objs[-1]])
    exe = str(out / "driver")
    _run([HIPCC, *objs, "-o", exe])
    return exe


def test_windows_of_the_row_forward_fit(driver):
    assert "rows: ok" in _run([driver, "rows"])


def test_windows_of_the_tile_adjoint_fit_and_hold_their_rays(driver):
    assert "tiles: ok" in _run([driver, "tiles"])


def test_adjoint_scratch_at_its_limits(driver):
    assert "scratch: ok" in _run([driver, "scratch"])


def test_dispatch(driver):
    assert "dispatch: ok" in _run([driver, "dispatch"])


def test_geometry_rules_look_at_the_columns_that_decide(driver):
    assert "columns: ok" in _run([driver, "columns"])


def test_geometry_creation_does_not_grow_with_the_columns():
    """720 views: sixteen times the columns at no more than four times the time (each
    view's rules look at a few columns; reading all of them grew sixteenfold)."""
    import time

    import paper_1609_00958_amd as gjp

    def best(n_u):
        v = gjp.views_circular_cone(720, 2048.0, 3072.0, 0.01, 1.0, n_u, 64)
        t = []
        for _ in range(9):
            t0 = time.perf_counter()
            gjp.Geometry((64, 64, 64), v, n_u, 64)
            t.append(time.perf_counter() - t0)
        return min(t)

    assert best(32000) < 4 * best(2000)
