"""The library's host side without a GPU: tests/native/fake_device.cpp stands in for
the HIP runtime and the kernel launchers, and is built with AddressSanitizer and
UndefinedBehaviorSanitizer, so that a launch that is handed freed memory ends the
program."""
import concurrent.futures as cf
import os
import shutil
import subprocess

import pytest

from tests.test_sanitize_native import CSRC, ROOT, SAN

SOURCES = ["geometry.cpp", "sphere_geometry.cpp", "schedule.cpp", "api_grid.cpp", "api_launch.cpp", "api_stencil.cpp",
           "api_ali.cpp", "api_krylov.cpp"]

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("fake_device")
    flags = ["-std=c++17", *SAN, "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
             "-I" + CSRC]

    def compile(src):
        obj = str(tmp / (os.path.basename(src) + ".o"))
        r = subprocess.run(["g++", *flags, "-c", src, "-o", obj], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr[-4000:]
        return obj

    files = [os.path.join(CSRC, f) for f in SOURCES] + [os.path.join(ROOT, "tests", "native", "fake_device.cpp")]
    with cf.ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(compile, files))
    exe = str(tmp / "fake_device")
    r = subprocess.run(["g++", *SAN, *objs, "-pthread", "-o", exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


def _case(fake, name):
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1:abort_on_error=0", UBSAN_OPTIONS="print_stacktrace=1")
    r = subprocess.run([fake, name], capture_output=True, text=True, timeout=300, env=env)
    assert r.returncode == 0 and f"{name} passed" in r.stdout, (r.stdout + r.stderr)[:4000]


def test_schedules_of_a_step_outlive_it(fake):
    """Solves whose batch shrinks at every step pass the 64 schedules that a grid
    keeps; the wavelength list and the Lambda* schedule that a step took at its
    beginning must not be freed by its later look-ups."""
    _case(fake, "shrinking_batches")


def test_schedules_of_many_calls(fake):
    """The same for formal solutions, direction subsets, stencils and BiCGStab."""
    _case(fake, "mixed_calls")


def test_short_memory_falls_back(fake):
    """Where the chosen shapes' partial sums or the stencil's tables do not fit, every
    call goes on with the default shapes and the kernel without tables."""
    _case(fake, "short_memory")


def test_default_shape_can_be_set_again(fake):
    """Also where a grid whose layers fit the LDS has band tiles for its default."""
    _case(fake, "default_shape_again")


def test_tuned_shape_can_be_set_again(fake):
    """Whichever shape the autotuner finds fastest, threads, rays and tile kind give it
    back on another grid, its number of bundles included."""
    _case(fake, "tuned_shape_again")


def test_shapes_are_asked_once(fake):
    """A call of a new size costs no queries to the runtime beyond the grid's first."""
    _case(fake, "shapes_asked_once")


def test_slots_of_a_schedule_are_bounded(fake):
    """By its workgroups and wavelengths per bundle, and by its items."""
    _case(fake, "slot_bound")


def test_routes_of_stencils(fake):
    """Where the templates of a quadrature cross two faces at once (45 degrees), the
    linear operator goes by rows as soon as the characteristics are many."""
    _case(fake, "stencil_routes")


def test_workgroups_of_a_cu_balance(fake):
    """Batches on several workgroups a CU: the heaviest shares of the wavelengths must
    not meet on one CU."""
    _case(fake, "balanced_cus")
