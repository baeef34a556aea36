"""Models at the edges of how the whole-iteration kernels share the work, each with the kernel that netmax_run takes for many iterations:
None where it launches the separate kernels.  test_launch_routes.py checks the kernel, test_gpu_small_iter.py the results."""
SMALL, SLICED, RESIDENT = "small_softmax_iteration_kernel", "sliced_softmax_kernel", "resident_mlp_kernel"

ONE_WORKGROUP = [(SMALL, over) for over in (
    # groups of draws: sixteen iterations, fifteen, five, one
    dict(M=3, dims=(20, 10), batch=64, n_per_worker=90), dict(M=3, dims=(21, 9), batch=65, n_per_worker=90), dict(M=2, dims=(6, 3), batch=200, n_per_worker=230),
    dict(M=2, dims=(3, 2), batch=600, n_per_worker=640),
    # peers counted by more than one wave, by every wave
    dict(M=65, dims=(24, 5), batch=9, n_per_worker=20), dict(M=256, dims=(12, 4), batch=4, n_per_worker=9),
    # matrix-instruction form: one, two and four row tiles; parts of one step, of odd and of even numbers of steps; few vectors and many
    dict(M=3, dims=(128, 10), batch=16, n_per_worker=40), dict(M=5, dims=(384, 16), batch=16, n_per_worker=40), dict(M=3, dims=(128, 7), batch=32, n_per_worker=40),
    dict(M=8, dims=(256, 10), batch=32, n_per_worker=40), dict(M=3, dims=(640, 3), batch=32, n_per_worker=40), dict(M=4, dims=(64, 16), batch=64, n_per_worker=80),
    dict(M=3, dims=(192, 2), batch=64, n_per_worker=80), dict(M=3, dims=(256, 10), batch=64, n_per_worker=80),
)]

SLICES = [(SLICED, over) for over in (
    # slices of seven steps (the waves of the last-layer kernel), four waves' and eight waves'; one row tile, two and four
    dict(M=16, dims=(784, 10), batch=64), dict(M=3, dims=(784, 10), batch=16), dict(M=2, dims=(512, 16), batch=64), dict(M=5, dims=(900, 3), batch=32),
    # a last slice of part of a step, of whole steps and a part, features that are a multiple of four only; batches that fill no row tile
    dict(M=3, dims=(788, 10), batch=64), dict(M=4, dims=(1020, 7), batch=33), dict(M=3, dims=(500, 10), batch=64), dict(M=3, dims=(900, 9), batch=9),
    # slices of eight steps
    dict(M=3, dims=(1024, 16), batch=50), dict(M=2, dims=(512, 10), batch=50),
    # as many workgroups as are resident: one a compute unit, seven slices
    dict(M=36, dims=(784, 10), batch=40),
)] + [
    # one worker more than that, and many more; slices of more than eight steps
    (None, dict(M=37, dims=(784, 10), batch=40)), (None, dict(M=73, dims=(784, 10), batch=40)), (None, dict(M=150, dims=(784, 10), batch=24)),
    (None, dict(M=2, dims=(1028, 16), batch=20)), (None, dict(M=4, dims=(1028, 7), batch=33)),
    # models of that many features that one workgroup holds
    (SMALL, dict(M=3, dims=(900, 2), batch=9)), (SMALL, dict(M=2, dims=(512, 5), batch=20)),
]

GROUPS_OF_UNITS = [(RESIDENT, over) for over in (
    # units of one workgroup, of several, of all compute units; both batches; strips of features that end inside, one per wave and four
    dict(M=3, dims=(64, 32, 10), batch=64), dict(M=2, dims=(8, 64, 3), batch=32), dict(M=5, dims=(264, 96, 16), batch=32), dict(M=16, dims=(784, 512, 10), batch=64),
    dict(M=9, dims=(784, 160, 10), batch=32), dict(M=3, dims=(856, 64, 2), batch=32), dict(M=2, dims=(200, 1024, 7), batch=64), dict(M=128, dims=(40, 64, 5), batch=32),
    # more units than words asked for together
    dict(M=4, dims=(96, 800, 10), batch=64), dict(M=3, dims=(96, 544, 10), batch=32), dict(M=3, dims=(64, 352, 4), batch=64),
)] + [
    # more workgroups than compute units; columns that do not fit LDS; few workgroups with much work each, where it does not pay
    (None, dict(M=17, dims=(96, 512, 10), batch=64)), (None, dict(M=2, dims=(1000, 64, 10), batch=32)), (None, dict(M=9, dims=(784, 160, 10), batch=64)),
]
