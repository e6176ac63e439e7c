"""Empty-space classification where a route between its kernels ends: a thread
per word (FP8, and bricks thin in y or x or of a few cells), rows of cells
dealt in long and in short runs, and tables long enough for a smaller grid.
All occupancy words against every cell's corners, through the brute force of
the per-cell test."""
import pytest

from test_gpu_classify_cells import test_every_cell as check_every_cell

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f32", "f16", "fp8"])
@pytest.mark.parametrize("dims,brick,K,op", [
    ((130, 5, 9), (130, 1, 9), 64, "composite"),            # 2 cells along y: 1 row of words in 16
    ((130, 21, 9), (130, 7, 9), 300, "mip"),                # 8 cells along y: 2 rows of words
    ((131, 22, 9), (131, 11, 9), 37, "composite"),          # 12 cells along y: 3 rows of words (FP16: 0.19 of the lanes)
    ((131, 30, 9), (131, 15, 9), 37, "composite"),          # 16 cells along y: 4 rows of words (0.25)
    ((3, 130, 67), (1, 130, 67), 256, "composite"),         # 2 cells along x
    ((33, 35, 37), (16, 16, 16), 1025, "mip"),              # small bricks, a long table
    ((32, 32, 32), (2, 2, 2), 1024, "composite"),           # 4096 bricks of 27 cells
    ((320, 320, 140), (20, 20, 20), 4096, "composite"),      # more words than a long table's grid takes at once
    ((90, 100, 80), (70, 80, 60), 1024, "composite"),       # bricks of different sizes: short runs
    ((90, 100, 80), (70, 80, 60), 4096, "mip"),
    ((256, 70, 300), (250, 66, 290), 100, "composite"),     # one large brick, the others slivers
])
def test_every_cell_at_the_edges_of_the_routes(storage, dims, brick, K, op):
    check_every_cell(storage, dims, brick, K, op)
