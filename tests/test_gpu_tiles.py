"""Edges of the pass kernels' tiles, against the oracle: sizes at which a tile
ends just before, exactly at or just beyond the domain's ring, and remainders
of one cell.  States must be bit-exact with the oracle in the run's type,
residuals within 1e-12 (FP64 sums of the same terms in another order)."""
import sys

import numpy as np
import pytest

import oracle
import synthetic
from gpu_util import bits_equal, oracle_residuals, oracle_run, run_device

pytestmark = pytest.mark.gpu

RNG = np.random.default_rng(77)


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def check(U0, f, h2, K, R, blocks, dtype, device, what, **tuning):
    want, b = oracle_run(U0, f, h2, K, dtype)
    ores, _ = oracle_residuals(np.asarray(U0, dtype=dtype), b, K, R)
    say(what)
    got, res = run_device(U0, f, h2, K, blocks, dtype, device, check_every=R, **tuning)
    assert bits_equal(got, want), what
    np.testing.assert_allclose(res, ores, rtol=1e-12, atol=0)


# 3D tiles hold 64 (FP32) / 32 (FP64) columns and 32 or 64 rows; k strips at
# depth 5 cover 56 k + 8 (FP32) or 24 k + 8 (FP64) columns, k row groups 24 k + 8
# or 56 k + 8 rows.
TILES_3D = [
    # (nx, ny, nz, bx, by, bz)
    (64, 64, 9, 2, 2, 2),     # one FP32 tile, exactly
    (120, 120, 6, 2, 3, 1),   # two, exactly
    (121, 119, 11, 3, 2, 2),  # one column beyond, one row short
    (32, 32, 21, 1, 2, 3),    # one 32-row tile, exactly
    (56, 88, 5, 2, 2, 1),     # two FP64 strips, exactly
    (57, 31, 7, 2, 1, 2),
    (65, 33, 1, 2, 2, 1),     # one plane
    (3, 65, 4, 1, 2, 2),
]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("case", TILES_3D)
def test_3d_tile_edges(device, dtype, case):
    nx, ny, nz, bx, by, bz = case
    U0 = RNG.uniform(0, 1, (nz + 2, ny + 2, nx + 2))
    f = RNG.uniform(-1, 1, (nz, ny, nx))
    h2 = synthetic.spacing2(max(nx, ny, nz))
    for src in (f, None):
        for depth, rows in ((0, 0), (5, 8), (4, 0), (2, 64)):
            check(U0, src, h2, 11, 5, (bx, by, bz), dtype, device,
                  "3d tiles %s %s depth %d rows %d" % (case, np.dtype(dtype).name, depth, rows),
                  depth=depth, rows=rows)
