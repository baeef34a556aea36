"""The kernels that netmax_run launches, and how, on the host code of the built library: tests/launch_routes_driver.cpp stands in for the runtime."""
import os
import shutil
import subprocess

import pytest

from paper_2009_05766_amd.build import LIB, build
from kernel_cases import ERRORS, FEW_CLASSES, FORWARD, RUNS, SAME_BITS
from whole_iteration_cases import GROUPS_OF_UNITS, ONE_WORKGROUP, RESIDENT, SLICED, SLICES, SMALL

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"), reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("routes") / "drive")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", os.path.join(ROOT, "tests", "launch_routes_driver.cpp"),
                    "-rdynamic", "-ldl", "-o", exe], check=True)
    lib = LIB if os.path.exists(LIB) else build()

    def forms(dims, M, batch, iters, offset=0, capture=0, cooperative=1, bf16=0, fused=0):
        """-> launches of one iteration by separate calls, launches of netmax_run: lists of (how, kernel, template arguments, workgroups)."""
        return drive([" ".join(str(int(v)) for v in (iters, M, batch, offset, capture, cooperative, bf16, fused, *dims))])[0][1:]

    def of(*a, **over):
        """The same as lists of (how, kernel)."""
        return [[launch[:2] for launch in part] for part in forms(*a, **over)]

    def drive(lines):
        r = subprocess.run([exe, lib], input="\n".join(lines), capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        return [[[tuple(launch.split(":")) for launch in part.split()] for part in line.split("|")] for line in r.stdout.splitlines()]
    of.drive, of.forms = drive, forms
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
             routes.drive(["9 4 50 0 0 1 0 0 100 50 10", "9 8 32 0 0 0 0 0 256 10", "9 16 64 0 0 1 0 0 784 10", "9 8 32 0 0 1 0 0 256 10"])]
    assert first == [[], [], [("cooperative", "no_work_kernel", "", "1")], []]


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


@pytest.mark.parametrize("M,batch,widths,strips", [
    # the rule's terms, one by one: a block's share of an XCD's rounds, two walks a compute unit, small batches, multiples of 64 workers
    (127, 128, (1152, 384), 2), (63, 128, (1664, 384), 4), (63, 128, (896, 128), 2), (63, 128, (384, 384), 1), (63, 128, (1024, 512), 8), (48, 128, (640, 640), 2),
    (8, 128, (1024, 1024), 4), (4, 128, (1024, 512), 1), (127, 64, (1152, 384), 1), (64, 128, (640, 384), 2), (64, 96, (1152, 896), 2), (128, 128, (1280, 512), 4),
    (128, 128, (3072, 1024), 8), (64, 128, (2944, 640), 4),
])
def test_walks_of_the_fused_weight_gradient(routes, M, batch, widths, strips):
    """The strips that a workgroup walks, from its launch's size."""
    launched = [int(groups) for _, kernel, _, groups in routes.forms((*widths, 10), M, batch, 1, bf16=1, fused=1)[1] if kernel == "wgrad_mix_mfma_kernel"]
    size = {walk: -(-(-(-widths[0] // 32 // walk)) * (widths[1] // 128) // 8) * 8 * M for walk in (1, 2, 4, 8)}
    assert launched == [size[strips]] and list(size.values()).count(size[strips]) == 1


@pytest.mark.parametrize("M,batch,dims,inside", [
    # few parameters in matrix-core layers; blocks that leave XCDs without work; walks of few strips; and where it pays
    (64, 128, (3000, 1000, 128, 128, 10), False), (64, 128, (2200, 384, 384, 10), False), (127, 128, (384, 128, 128, 10), False), (48, 128, (640, 640, 10), True),
    # small states, whose operands and peers come from the last cache
    (48, 128, (384, 384, 10), True), (18, 128, (128, 1536, 3), True), (41, 128, (128, 512, 23), True),
    (64, 128, (784, 384, 384, 10), False), (64, 128, (1000, 512, 512, 10), True), (64, 128, (200, 1024, 1024, 10), True), (48, 128, (3072, 1024, 1024, 10), True),
    (32, 64, (1024, 1024, 10), True), (64, 64, (640, 384, 10), True), (100, 32, (1152, 384, 10), True), (5, 32, (512, 512, 128, 10), False),
])
def test_update_in_matrix_core_weight_gradients(routes, M, batch, dims, inside):
    """Iterations of netmax_run that another follows: the weight gradients of matrix-core layers update their columns where that saves bytes."""
    run = [kernel for _, kernel in routes(dims, M, batch, 3, bf16=1)[1]]
    first = run[:run.index("mix_subset_kernel" if inside else "mix_kernel") + 1]
    assert ("wgrad_mix_mfma_kernel" in first) == inside and ("wgrad_mfma_kernel" in first) != inside


@pytest.mark.parametrize("M,batch,dims,inside", [
    # an iteration that leaves g: many workers, many more of them, blocks and operands that eat up what is saved
    (127, 128, (1024, 1024, 10), True), (128, 128, (3072, 1024, 1024, 10), False), (128, 64, (1024, 1024, 10), False), (191, 32, (512, 512, 256, 10), True), (192, 32, (512, 512, 256, 10), False),
    (256, 64, (1024, 1024, 10), False), (127, 128, (384, 384, 10), False), (122, 96, (640, 640, 10), False), (64, 64, (512, 384, 128, 10), True), (14, 128, (256, 256, 896, 16), True), (48, 128, (784, 384, 384, 10), False), (96, 64, (3072, 512, 512, 10), True),
])
def test_update_in_the_last_iteration(routes, M, batch, dims, inside):
    run = [kernel for _, kernel in routes(dims, M, batch, 1, bf16=1)[1]]
    assert ("wgrad_mix_mfma_kernel" in run) == inside and ("mix_kernel" in run) != inside


def _local_step(routes, operands, M, batch, dims):
    """Kernels of a gradient, with their template arguments."""
    return ["%s<%s>" % launch[1:3] for launch in routes.forms(dims, M, batch, 1, bf16=operands == "bf16")[0]]


def test_layer_cases_reach_their_kernel(routes):
    for operands, M, batch, dims, kernel in FORWARD:
        assert next(k for k in _local_step(routes, operands, M, batch, dims) if "fwd" in k) == kernel, (operands, M, batch, dims)
    for operands, M, batch, dims, kernel in ERRORS:                  # from the last layer down: the second layer's comes last
        assert [k for k in _local_step(routes, operands, M, batch, dims) if "dgrad" in k][-1] == kernel, (operands, M, batch, dims)
    for M, batch, dims, kernel in FEW_CLASSES:
        assert [k for k in _local_step(routes, "bf16", M, batch, dims) if "fwd_small" in k] == [kernel], (M, batch, dims)
    reached = {c[-1] for c in FORWARD + ERRORS}
    assert len([k for k in reached if "wave_fwd" in k]) == 16 and len([k for k in reached if "chain_fwd" in k]) == 5
    assert len([k for k in reached if "wave_dgrad" in k]) == 12 and len([k for k in reached if "chain_dgrad" in k]) == 13


def test_few_and_many_workers_differ_in_these_kernels(routes):
    for few, many, batch, dims, among_few, among_many, _ in SAME_BITS:
        pairs = list(zip(*(_local_step(routes, "bf16", M, batch, dims) for M in (few, many))))
        assert [" ".join(k) for k in zip(*(p for p in pairs if p[0] != p[1]))] == [among_few, among_many], (few, many, batch, dims)


@pytest.mark.parametrize("M,batch,dims,followed,last", RUNS)
def test_runs_reach_the_update_in_weight_gradients(routes, M, batch, dims, followed, last):
    run = [kernel for _, kernel in routes(dims, M, batch, 2, bf16=1)[1]]
    half = (len(run) + 1) // 2 if followed == last else run.index("mix_subset_kernel" if followed else "mix_kernel") + 1
    assert ("wgrad_mix_mfma_kernel" in run[:half]) == followed and ("wgrad_mix_mfma_kernel" in run[half:]) == last
