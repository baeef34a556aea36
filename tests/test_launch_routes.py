"""The kernels that netmax_run launches, and how, on the host code of the built library: tests/launch_routes_driver.cpp stands in for the runtime."""
import os
import shutil
import subprocess

import pytest

from paper_2009_05766_amd.build import LIB, build
from whole_iteration_cases import GROUPS_OF_UNITS, ONE_WORKGROUP, RESIDENT, SLICED, SLICES, SMALL

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"), reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("routes") / "drive")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", os.path.join(ROOT, "tests", "launch_routes_driver.cpp"),
                    "-rdynamic", "-ldl", "-o", exe], check=True)
    lib = LIB if os.path.exists(LIB) else build()

    def of(dims, M, batch, iters, offset=0, capture=0, cooperative=1):
        """-> launches of one iteration by separate calls, launches of netmax_run: lists of (how, kernel)."""
        return drive([" ".join(str(v) for v in (iters, M, batch, offset, capture, cooperative, *dims))])[0][1:]

    def drive(lines):
        r = subprocess.run([exe, lib], input="\n".join(lines), capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return [[[tuple(launch.split(":")) for launch in part.split()] for part in line.split("|")] for line in r.stdout.splitlines()]
    of.drive = drive
    return of


@pytest.mark.parametrize("dims,M,batch,kernel,few,many", [((256, 10), 8, 32, SMALL, 7, 8), ((21, 9), 3, 65, SMALL, 2, 30), ((784, 10), 16, 64, SLICED, 4, 5),
                                                          ((1024, 16), 3, 50, SLICED, 1, 9), ((784, 512, 10), 16, 64, RESIDENT, 1, 2),
                                                          ((64, 32, 10), 3, 64, RESIDENT, 2, 18)])
def test_launches_that_wait_are_cooperative(routes, dims, M, batch, kernel, few, many):
    """Workgroups that wait for each other in a plain launch may hold compute units that the missing ones, or another process's, need."""
    calls, run = routes(dims, M, batch, many)
    assert run == [("cooperative", kernel)] and all(how == "plain" for how, _ in calls)
    run = routes(dims, M, batch, few)[1]
    assert len(run) > 1 and all(how == "plain" for how, _ in run)
    # nothing that waits where the promise is not to be had: a stream under capture, a device without such launches
    for over in (dict(capture=1), dict(cooperative=0)):
        run = routes(dims, M, batch, many, **over)[1]
        assert len(run) >= many and all(how == "plain" and (name == SMALL) == (kernel == SMALL) for how, name in run)


def test_first_cooperative_launch_of_a_process(routes):
    """It takes milliseconds and belongs to preparation; contexts that make no such launches do without, further ones do not repeat it."""
    first = [[launch for launch in parts[0] if launch[0] == "cooperative"] for parts in
             routes.drive(["9 4 50 0 0 1 100 50 10", "9 8 32 0 0 0 256 10", "9 16 64 0 0 1 784 10", "9 8 32 0 0 1 256 10"])]
    assert first == [[], [], [("cooperative", "no_work_kernel")], []]


@pytest.mark.parametrize("dims,M,batch", [((784, 10), 37, 64), ((784, 512, 10), 17, 64), ((256, 10), 257, 32)])
def test_more_workgroups_than_fit(routes, dims, M, batch):
    assert all(how == "plain" for how, _ in routes(dims, M, batch, 20)[1])


@pytest.mark.parametrize("offset", [0, 4, 8, 12, 16])
def test_features_that_start_anywhere(routes, offset):
    """The resident kernel adds the hidden layer's products as fwd_f32_kernel does; where the separate calls take another forward kernel because the
    features do not start at a multiple of 16 bytes, netmax_run takes that one, too."""
    calls, run = routes((784, 512, 10), 16, 64, 8, offset=offset)
    if offset % 16 == 0:
        assert ("plain", "fwd_f32_kernel") in calls and run == [("cooperative", RESIDENT)]
    else:
        forward = calls[2]
        assert forward[1] not in ("fwd_f32_kernel", RESIDENT) and run.count(forward) == 8 and all(how == "plain" for how, _ in run)


@pytest.mark.parametrize("kernel,over", ONE_WORKGROUP + SLICES + GROUPS_OF_UNITS)
def test_cases_reach_their_kernel(routes, kernel, over):
    run = routes(over["dims"], over["M"], over["batch"], 18)[1]
    if kernel:
        assert run == [("cooperative", kernel)]
    else:
        assert all(how == "plain" and name not in (SMALL, SLICED, RESIDENT) for how, name in run)
