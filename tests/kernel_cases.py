"""Networks at the edges of the kernels for few blocks and of the update inside weight gradients, each with the kernel that it is there for.
test_launch_routes.py checks the kernels on the host code, test_gpu_tile_layers.py and test_gpu_run_update.py the results."""

# Forward pass: (operands, workers, batch, dims, kernel of the first layer).  wave_fwd_kernel<bfloat16, row tiles, tail, steps ahead, far rows>
FORWARD = [
    # whole steps of sixteen indices (bfloat16 32), one more, one fewer, contractions of less than a step; two and three steps ahead
    ("f32", 2, 31, (640, 33, 10), "wave_fwd_kernel<false,1,false,2,false>"), ("f32", 3, 33, (641, 65, 10), "wave_fwd_kernel<false,1,true,2,false>"),
    ("f32", 9, 129, (655, 68, 10), "wave_fwd_kernel<false,1,true,2,false>"), ("f32", 2, 20, (1000, 40), "wave_fwd_kernel<false,1,true,2,false>"),
    ("f32", 3, 3, (3, 34, 10), "wave_fwd_kernel<false,1,true,2,false>"), ("f32", 2, 40, (1030, 33, 10), "wave_fwd_kernel<false,1,true,3,false>"),
    ("f32", 3, 20, (1040, 36, 10), "wave_fwd_kernel<false,1,false,3,false>"),
    ("bf16", 2, 31, (640, 33, 10), "wave_fwd_kernel<true,1,false,2,false>"), ("bf16", 3, 33, (641, 65, 10), "wave_fwd_kernel<true,1,true,2,false>"),
    ("bf16", 9, 129, (671, 68, 10), "wave_fwd_kernel<true,1,true,2,false>"), ("bf16", 2, 20, (1000, 40), "wave_fwd_kernel<true,1,true,2,false>"),
    # two and four tiles of 32 batch rows
    ("f32", 5, 40, (400, 960, 10), "wave_fwd_kernel<false,2,false,2,false>"), ("f32", 5, 50, (401, 957, 10), "wave_fwd_kernel<false,2,true,2,false>"),
    ("f32", 5, 40, (1040, 960, 10), "wave_fwd_kernel<false,2,false,3,false>"), ("f32", 5, 60, (1031, 957, 10), "wave_fwd_kernel<false,2,true,3,false>"),
    ("bf16", 5, 40, (416, 960, 10), "wave_fwd_kernel<true,2,false,2,false>"), ("bf16", 5, 60, (400, 957, 10), "wave_fwd_kernel<true,2,true,2,false>"),
    ("bf16", 5, 100, (416, 960, 10), "wave_fwd_kernel<true,4,false,2,false>"), ("bf16", 5, 97, (401, 957, 10), "wave_fwd_kernel<true,4,true,2,false>"),
    # rows of W beyond 32-bit offsets (a batch in which the one rounding that falls the other way is one of hundreds of activations)
    ("f32", 2049, 31, (3, 36, 3), "wave_fwd_kernel<false,1,true,2,true>"), ("bf16", 2049, 31, (3, 36, 3), "wave_fwd_kernel<true,1,true,2,true>"),
    # one chain.  Aligned layers (both orientations of the activations): fewer steps than waves, one, two and four row tiles
    ("bf16", 3, 32, (128, 128, 10), "chain_fwd_kernel<1,false>"), ("bf16", 2, 64, (256, 384, 128, 10), "chain_fwd_kernel<2,false>"),
    ("bf16", 17, 96, (1280, 256, 10), "chain_fwd_kernel<4,false>"),
    # others, two parts of a batch among them
    ("bf16", 32, 60, (672, 500, 10), "chain_fwd_kernel<2,false>"), ("bf16", 32, 33, (641, 511, 10), "chain_fwd_kernel<2,true>"),
    ("bf16", 16, 100, (800, 500, 10), "chain_fwd_kernel<4,false>"), ("bf16", 8, 250, (650, 510, 10), "chain_fwd_kernel<4,true>"),
    # a general layer under aligned ones
    ("bf16", 2, 128, (700, 128, 128, 10), "wave_fwd_kernel<true,1,true,2,false>"),
    # the most blocks that each takes, and one worker more
    ("f32", 42, 65, (640, 500, 10), "wave_fwd_kernel<false,1,false,2,false>"), ("f32", 43, 65, (640, 500, 10), "split_fwd_kernel<true>"),
    ("f32", 20, 33, (644, 1024, 10), "wave_fwd_kernel<false,1,true,2,false>"), ("f32", 21, 33, (644, 1024, 10), "tile_fwd_kernel<false,true,64,64,64,2,2>"),
    ("f32", 68, 20, (100, 900, 10), "wave_fwd_kernel<false,1,true,2,false>"), ("f32", 69, 20, (100, 900, 10), "tile_fwd_kernel<false,true,32,64,64,1,2>"),
    ("bf16", 31, 20, (640, 1024, 10), "wave_fwd_kernel<true,1,false,2,false>"), ("bf16", 32, 20, (640, 1024, 10), "tile_fwd_kernel<true,true,32,64,64,1,2>"),
    ("bf16", 10, 65, (640, 1020, 10), "wave_fwd_kernel<true,1,false,2,false>"), ("bf16", 11, 65, (640, 1020, 10), "tile_fwd_kernel<true,true,128,32,128,4,1>"),
    ("bf16", 33, 60, (672, 500, 10), "tile_fwd_kernel<true,true,64,64,128,2,2>"), ("bf16", 17, 100, (800, 500, 10), "tile_fwd_kernel<true,true,128,32,128,4,1>"),
    ("bf16", 24, 32, (384, 1024, 10), "chain_fwd_kernel<1,false>"), ("bf16", 25, 32, (384, 1024, 10), "fwd_mfma_kernel<true>"),
    ("bf16", 32, 32, (1024, 1024, 10), "chain_fwd_kernel<1,false>"), ("bf16", 33, 32, (1024, 1024, 10), "fwd_mfma_kernel<true>"),
    ("bf16", 16, 64, (512, 1024, 10), "chain_fwd_kernel<2,false>"), ("bf16", 17, 64, (512, 1024, 10), "fwd_mfma_kernel<true>"),
    ("bf16", 16, 128, (384, 1024, 10), "chain_fwd_kernel<4,false>"), ("bf16", 17, 128, (384, 1024, 10), "fwd_mfma_kernel<true>"),
]

# Errors of hidden layers: (operands, workers, batch, dims, kernel of the second layer's).  wave_dgrad_kernel<row tiles, pieces of W aligned, tail>,
# chain_dgrad_kernel<aligned layer, row tiles, pieces of W aligned, tail>
ERRORS = [
    # whole steps of sixteen outputs (bfloat16 32), one more, fewer than a step; rows of W that start anywhere
    ("f32", 2, 31, (20, 33, 160, 10), "wave_dgrad_kernel<1,false,false>"), ("f32", 2, 20, (20, 40, 7, 33, 10), "wave_dgrad_kernel<1,false,true>"),
    ("f32", 3, 20, (20, 36, 48, 10), "wave_dgrad_kernel<1,true,false>"), ("f32", 3, 9, (20, 36, 44, 10), "wave_dgrad_kernel<1,true,true>"),
    ("f32", 3, 33, (20, 65, 129, 10), "wave_dgrad_kernel<2,false,true>"), ("f32", 2, 64, (21, 31, 34, 10), "wave_dgrad_kernel<2,false,true>"),
    ("f32", 3, 40, (21, 35, 48, 10), "wave_dgrad_kernel<2,false,false>"), ("f32", 3, 40, (20, 36, 48, 10), "wave_dgrad_kernel<2,true,false>"),
    ("f32", 2, 100, (20, 36, 656, 10), "wave_dgrad_kernel<4,true,false>"), ("f32", 3, 97, (20, 36, 644, 10), "wave_dgrad_kernel<4,true,true>"),
    ("f32", 2, 128, (21, 35, 643, 10), "wave_dgrad_kernel<4,false,true>"), ("f32", 2, 150, (21, 35, 643, 10), "wave_dgrad_kernel<4,false,true>"),
    ("f32", 3, 65, (21, 35, 80, 10), "wave_dgrad_kernel<4,false,false>"),
    ("bf16", 3, 20, (21, 301, 1001, 10), "chain_dgrad_kernel<false,1,false,true>"), ("bf16", 2, 31, (21, 35, 288, 10), "chain_dgrad_kernel<false,1,false,false>"),
    ("bf16", 2, 20, (20, 100, 1000, 10), "chain_dgrad_kernel<false,1,true,true>"), ("bf16", 2, 20, (20, 100, 672, 10), "chain_dgrad_kernel<false,1,true,false>"),
    ("bf16", 3, 60, (21, 301, 1001, 10), "chain_dgrad_kernel<false,2,false,true>"), ("bf16", 2, 33, (21, 35, 288, 10), "chain_dgrad_kernel<false,2,false,false>"),
    ("bf16", 2, 60, (20, 100, 1000, 10), "chain_dgrad_kernel<false,2,true,true>"), ("bf16", 2, 60, (20, 100, 672, 10), "chain_dgrad_kernel<false,2,true,false>"),
    ("bf16", 3, 100, (21, 301, 1001, 10), "chain_dgrad_kernel<false,4,false,true>"), ("bf16", 2, 128, (21, 35, 288, 10), "chain_dgrad_kernel<false,4,false,false>"),
    # the kernel of any number of blocks
    ("bf16", 2, 31, (20, 33, 160, 10), "tile_dgrad_kernel<true,false,32,64,64,1,2>"), ("bf16", 3, 33, (20, 65, 129, 10), "tile_dgrad_kernel<true,false,64,64,128,2,2>"),
    # aligned layers over general and aligned ones: fewer steps than waves and more, one, two and four row tiles
    ("bf16", 2, 32, (60, 128, 128, 10), "chain_dgrad_kernel<true,1,true,false>"), ("bf16", 2, 64, (128, 256, 384, 10), "chain_dgrad_kernel<true,2,true,false>"),
    ("bf16", 3, 96, (100, 128, 512, 10), "chain_dgrad_kernel<true,4,true,false>"), ("bf16", 2, 128, (128, 128, 128, 40), "chain_dgrad_kernel<true,4,true,false>"),
    ("bf16", 2, 64, (100, 100, 128, 128, 10), "tile_dgrad_kernel<true,true,64,64,128,2,2>"),
    # the most blocks that each takes, and one worker more
    ("f32", 48, 20, (20, 1000, 30, 10), "wave_dgrad_kernel<1,false,true>"), ("f32", 49, 20, (20, 1000, 30, 10), "tile_dgrad_kernel<false,false,32,64,64,1,2>"),
    ("f32", 64, 40, (20, 128, 40, 10), "wave_dgrad_kernel<2,true,true>"), ("f32", 65, 40, (20, 128, 40, 10), "tile_dgrad_kernel<false,true,64,64,64,2,2>"),
    ("f32", 16, 40, (20, 1024, 640, 10), "wave_dgrad_kernel<2,true,false>"), ("f32", 17, 40, (20, 1024, 640, 10), "tile_dgrad_kernel<false,true,64,64,64,2,2>"),
    ("f32", 32, 40, (21, 1023, 259, 10), "wave_dgrad_kernel<2,false,true>"), ("f32", 33, 40, (21, 1023, 259, 10), "tile_dgrad_kernel<false,false,64,64,64,2,2>"),
    ("f32", 8, 65, (20, 1024, 640, 10), "wave_dgrad_kernel<4,true,false>"), ("f32", 9, 65, (20, 1024, 640, 10), "tile_dgrad_kernel<false,true,128,64,64,2,2>"),
    ("f32", 16, 65, (21, 1023, 481, 10), "wave_dgrad_kernel<4,false,true>"), ("f32", 17, 65, (21, 1023, 481, 10), "tile_dgrad_kernel<false,false,128,64,64,2,2>"),
    ("f32", 8, 65, (21, 1023, 67, 10), "wave_dgrad_kernel<4,false,true>"), ("f32", 9, 65, (21, 1023, 67, 10), "tile_dgrad_kernel<false,false,128,64,64,2,2>"),
    ("bf16", 64, 32, (20, 1024, 128, 10), "chain_dgrad_kernel<true,1,true,false>"), ("bf16", 65, 32, (20, 1024, 128, 10), "dgrad_mfma_kernel<>"),
    ("bf16", 48, 64, (20, 1024, 128, 10), "chain_dgrad_kernel<true,2,true,false>"), ("bf16", 49, 64, (20, 1024, 128, 10), "dgrad_mfma_kernel<>"),
    ("bf16", 24, 96, (20, 1024, 128, 10), "chain_dgrad_kernel<true,4,true,false>"), ("bf16", 25, 96, (20, 1024, 128, 10), "dgrad_mfma_kernel<>"),
    ("bf16", 16, 20, (21, 1023, 259, 10), "chain_dgrad_kernel<false,1,false,true>"), ("bf16", 17, 20, (21, 1023, 259, 10), "tile_dgrad_kernel<true,false,32,64,64,1,2>"),
    ("bf16", 16, 20, (20, 1000, 640, 10), "chain_dgrad_kernel<false,1,true,false>"), ("bf16", 17, 20, (20, 1000, 640, 10), "tile_dgrad_kernel<true,true,32,64,64,1,2>"),
    ("bf16", 8, 60, (20, 1000, 640, 10), "chain_dgrad_kernel<false,2,true,false>"), ("bf16", 9, 60, (20, 1000, 640, 10), "tile_dgrad_kernel<true,true,64,64,128,2,2>"),
]

# bfloat16 networks of few and of many workers that differ in one or two kernels only: (few, many, batch, dims, kernels among few, those among many in
# whose order they add, whether the column sums are added in that order, too)
SAME_BITS = [
    # aligned layers, forward and error: one, two, three and four row tiles, fewer steps than a chunk, a start of the contraction of every kind
    (3, 70, 32, (128, 1024, 256, 10), "chain_fwd_kernel<1,false> chain_dgrad_kernel<true,1,true,false>", "fwd_mfma_kernel<true> dgrad_mfma_kernel<>", True),
    (5, 52, 64, (384, 1024, 128, 10), "chain_fwd_kernel<2,false> chain_dgrad_kernel<true,2,true,false>", "fwd_mfma_kernel<true> dgrad_mfma_kernel<>", True),
    (4, 30, 96, (256, 1024, 384, 10), "chain_fwd_kernel<4,false> chain_dgrad_kernel<true,4,true,false>", "fwd_mfma_kernel<true> dgrad_mfma_kernel<>", True),
    (9, 30, 128, (1280, 1024, 128, 40), "chain_fwd_kernel<4,false> chain_dgrad_kernel<true,4,true,false>", "fwd_mfma_kernel<true> dgrad_mfma_kernel<>", True),
    # a general layer below (of less than a step: one part, whichever kernel) and above; a second aligned layer
    (3, 70, 32, (24, 1024, 128, 100, 10), "wave_fwd_kernel<true,1,true,2,false> chain_dgrad_kernel<true,1,true,false>", "tile_fwd_kernel<true,true,32,64,64,1,2> dgrad_mfma_kernel<>", True),
    (3, 30, 96, (100, 128, 1024, 10), "chain_fwd_kernel<4,false>", "fwd_mfma_kernel<false>", True),
    # layers of any width in one chain: whole steps and what is behind them, rows and columns that fill no block
    (16, 18, 100, (800, 500, 10), "chain_fwd_kernel<4,false>", "tile_fwd_kernel<true,true,128,32,128,4,1>", True),
    (16, 18, 100, (649, 497, 10), "chain_fwd_kernel<4,true>", "tile_fwd_kernel<true,false,128,32,128,4,1>", True),
    (32, 34, 60, (672, 500, 10), "chain_fwd_kernel<2,false>", "tile_fwd_kernel<true,true,64,64,128,2,2>", True),
    (32, 34, 33, (641, 511, 10), "chain_fwd_kernel<2,true>", "tile_fwd_kernel<true,false,64,64,128,2,2>", True),
    # their errors: rows of W aligned and not, tails.  Beyond 64 rows the other kernel's column sums change with the number of blocks
    (16, 17, 20, (20, 1000, 640, 10), "chain_dgrad_kernel<false,1,true,false>", "tile_dgrad_kernel<true,true,32,64,64,1,2>", True),
    (16, 17, 31, (20, 1000, 644, 10), "chain_dgrad_kernel<false,1,true,true>", "tile_dgrad_kernel<true,true,32,64,64,1,2>", True),
    (8, 9, 60, (20, 1000, 640, 10), "chain_dgrad_kernel<false,2,true,false>", "tile_dgrad_kernel<true,true,64,64,128,2,2>", True),
    (8, 9, 40, (20, 1000, 644, 10), "chain_dgrad_kernel<false,2,true,true>", "tile_dgrad_kernel<true,true,64,64,128,2,2>", True),
    (16, 17, 20, (21, 1023, 259, 10), "chain_dgrad_kernel<false,1,false,true>", "tile_dgrad_kernel<true,false,32,64,64,1,2>", True),
    (16, 17, 60, (21, 1023, 288, 10), "chain_dgrad_kernel<false,2,false,false>", "tile_dgrad_kernel<true,false,64,64,128,2,2>", True),
    (16, 17, 100, (21, 1023, 259, 10), "tile_fwd_kernel<true,false,128,32,128,4,1> chain_dgrad_kernel<false,4,false,true>",
     "tile_fwd_kernel<true,false,128,64,64,2,2> tile_dgrad_kernel<true,false,128,64,64,2,2>", False),
    (16, 17, 128, (21, 1023, 288, 10), "tile_fwd_kernel<true,false,128,32,128,4,1> chain_dgrad_kernel<false,4,false,false>",
     "tile_fwd_kernel<true,false,128,64,64,2,2> tile_dgrad_kernel<true,false,128,64,64,2,2>", False),
]

# Last layer of the matrix-core path: (workers, batch, dims, its forward kernel).  fwd_small_mfma_kernel<pieces ahead, workgroups that fit a compute unit's registers>
FEW_CLASSES = [
    # two pieces of 64 features, one group of four and two left over, the most (32); one to four waves, classes on either side of the columns of a
    # matrix instruction
    (3, 32, (128, 128, 2), "fwd_small_mfma_kernel<4,3>"), (2, 64, (64, 384, 17), "fwd_small_mfma_kernel<4,3>"), (3, 96, (40, 128, 32), "fwd_small_mfma_kernel<4,3>"),
    (2, 128, (128, 384, 31), "fwd_small_mfma_kernel<4,3>"), (2, 128, (36, 2048, 10), "fwd_small_mfma_kernel<4,3>"), (5, 32, (36, 2048, 32), "fwd_small_mfma_kernel<4,3>"),
    # the most workers in a round of three workgroups a compute unit and one more; in rounds of three and four alike; what LDS leaves no room for
    (768, 32, (36, 128, 3), "fwd_small_mfma_kernel<4,3>"), (769, 32, (36, 128, 3), "fwd_small_mfma_kernel<2,4>"), (800, 96, (36, 384, 2), "fwd_small_mfma_kernel<2,4>"),
    (1025, 32, (36, 128, 3), "fwd_small_mfma_kernel<4,3>"), (769, 64, (36, 512, 32), "fwd_small_mfma_kernel<4,3>"),
]

# netmax_run of bfloat16 networks with matrix-core layers: (workers, batch, dims, whether their weight gradients update their columns in an iteration that
# another follows, and in one that leaves g)
RUNS = [
    # 1.8 million floats, from which on they may: either side; one strip of 32 rows a walk
    (6, 32, (512, 512, 128, 10), True, True), (5, 32, (512, 512, 128, 10), False, False), (14, 64, (130, 256, 384, 10), True, True), (9, 64, (1024, 512), True, True),
    # walks of one strip, of two, four and eight, whole and with four left over, from the first strip and from a later one, of the first layer and of another
    (20, 128, (512, 512, 384, 10), True, True), (48, 128, (640, 640, 10), True, False), (48, 128, (1024, 1024, 10), True, True), (64, 128, (1024, 1024, 10), True, True), (7, 128, (2944, 1024, 10), True, True),
    (7, 128, (128, 2944, 1024, 10), True, True), (64, 96, (1664, 1024, 128, 10), True, True), (128, 128, (128, 896, 640, 10), True, False),
    # blocks that are no whole rounds over the XCDs
    (40, 128, (1152, 384, 10), True, False),
]
