"""HIP path vs the CPU oracle at the sizes where a kernel's tiles, capacities
or dispatch rules change over, bit-exact (see tests/test_gpu_parity.py)."""
import numpy as np
import pytest

from paper_1912_02984_amd import workloads as W
from tests.test_gpu_parity import run_both

pytestmark = pytest.mark.gpu


def _points_in(lin, dims, rng):
    """A point at a random place well inside each 0.1-sized voxel of `lin`."""
    g = np.stack([lin % dims[0], lin // dims[0] % dims[1], lin // (dims[0] * dims[1])], -1)
    return ((g + rng.uniform(0.1, 0.9, g.shape)) * 0.1).astype(np.float32)


@pytest.mark.parametrize("order", ["shuffled", "by brick"])
@pytest.mark.parametrize("words,depth", [(4, 64), (8, 128), (16, 256), (32, 300)])
def test_brick_sizes(words, depth, order):
    """The brick build with 4 to 32 occupancy words a brick: bricks of 256
    points (one wave) and 257 (a block), of 4096 (one part) and 4097 (two), a
    brick of three voxels with 9000 points whose later parts lie wholly past
    the cap, an empty first brick and a last brick cut short or full; with the
    points shuffled over the sort tiles and with whole tiles in one brick."""
    rng = np.random.default_rng(words)
    dims = (64, 64, depth)
    V, bv = dims[0] * dims[1] * dims[2], 64 * words
    lin = [np.array([V - 1] * 70)]
    for brick, n in ((1, 256), (2, 257), (4, 4096), (5, 4097)):
        lin.append(brick * bv + rng.integers(0, bv, n))
    lin.append(7 * bv + rng.choice([0, 17, bv - 1], 9000, p=[0.1, 0.7, 0.2]))
    lin.append(rng.integers(9 * bv, V, 2000))
    lin = np.concatenate(lin)
    P = np.stack([_points_in(lin, dims, rng) for _ in range(2)])
    if order == "shuffled":
        P = P[:, rng.permutation(P.shape[1])]
    for n_v in (1, 64):
        spec = W.GridSpec((0.0,) * 3, (0.1,) * 3, dims, n_v, 1)
        run_both(P, spec, 500, 32, "rvs", "knn", 3, where=f"words={words} n_v={n_v} {order}")
