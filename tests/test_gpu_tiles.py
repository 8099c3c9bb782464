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


# 2D tiles held in registers: 64 x 32, 64 x 64, 128 x 64, 128 x 128 and (FP32)
# 256 x 128 cells, picked by grid size; a pass of t sweeps loses t rows and t
# columns (rounded up to a lane's columns) on the sides without a ring.
TILES_2D = [
    # (nx, ny, bx, by, sweeps per pass)
    (64, 32, 2, 2, 8),      # one tile, exactly
    (65, 33, 2, 3, 8),
    (112, 48, 3, 2, 8),     # two strips and two groups, exactly
    (113, 47, 2, 2, 8),
    (63, 31, 1, 1, 13),
    (1, 1, 1, 1, 5),
    (3, 200, 1, 5, 12),
    (300, 3, 4, 1, 16),
    (517, 300, 5, 4, 16),
    (1000, 777, 4, 3, 13),
    (1502, 1499, 6, 5, 13),
    (2049, 2030, 8, 8, 16),
]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("case", TILES_2D)
def test_2d_register_tiles(device, dtype, case):
    nx, ny, bx, by, t = case
    U0 = RNG.uniform(0, 1, (ny + 2, nx + 2))
    f = RNG.standard_normal((ny, nx)) * 100
    h2 = synthetic.spacing2(max(nx, ny))
    for src in (f, None):
        for K, R in ((2 * t + 1, t), (3, 2)):
            check(U0, src, h2, K, R, (bx, by), dtype, device,
                  "2d tiles %s %s source %s" % (case, np.dtype(dtype).name, src is not None))


@pytest.mark.parametrize("case", [(64, 32, 2, 2, 26), (113, 47, 2, 2, 9), (700, 301, 3, 2, 16),
                                  (1030, 1101, 4, 5, 31), (2, 3, 1, 1, 33)])
def test_adjoint_register_tiles(device, case):
    """FP64 adjoint bit-exact with the oracle's (the accumulator adds the
    levels in the same order), whatever the passes."""
    import torch
    import paper_2303_02543_amd as jb
    nx, ny, bx, by, K = case
    h2 = synthetic.spacing2(max(nx, ny))
    full = RNG.standard_normal((ny + 2, nx + 2))
    Gb, dU0 = oracle.adjoint2d_full(full, K)
    s = jb.Solver((nx, ny), (bx, by), torch.float64, device=device)
    try:
        for chunk in (None, 7):
            say("adjoint tiles", case, chunk)
            gf, gU0 = s.adjoint(torch.from_numpy(full).to(device), K, h2, chunk=chunk)
            assert bits_equal(gf.cpu().numpy(), h2 * Gb)
            assert bits_equal(gU0.cpu().numpy(), dU0)
    finally:
        s.close()


# FP64 passes of up to four sweeps on the row kernel: depth 4 where its rounds
# are the shorter ones (256^3), depths 1 - 3 from 2^26 cells on.
ROWS_3D = [
    # (nx, ny, nz, bx, by, bz, depth, z segment)
    (256, 256, 256, 4, 4, 4, 4, 0),
    (251, 263, 259, 3, 4, 2, 4, 0),
    (512, 512, 256, 8, 8, 4, 1, 0),
    (419, 401, 403, 3, 4, 5, 2, 0),
    (419, 401, 403, 4, 3, 2, 3, 37),
]


@pytest.mark.parametrize("case", ROWS_3D)
def test_3d_rows(device, case):
    nx, ny, nz, bx, by, bz, depth, zseg = case
    rng = np.random.default_rng(5)
    U0 = rng.uniform(0, 1, (nz + 2, ny + 2, nx + 2))
    f = rng.uniform(-1, 1, (nz, ny, nx))
    h2 = synthetic.spacing2(max(nx, ny, nz))
    for src in (f, None):
        check(U0, src, h2, 4, 3, (bx, by, bz), np.float64, device,
              "3d rows %s %s" % (case, "laplace" if src is None else "poisson"),
              depth=depth, rows=zseg)


@pytest.mark.parametrize("src", [False, True])
def test_3d_rows_residual_alone(device, src):
    """The residual of a large FP64 grid by itself: the row kernel without stores."""
    import torch
    import paper_2303_02543_amd as jb
    grid, blocks = (300, 299, 321), (3, 3, 3)
    shape = tuple(reversed(grid))
    rng = np.random.default_rng(12)
    U = rng.uniform(0, 1, tuple(n + 2 for n in shape))
    f = rng.uniform(-1, 1, shape)
    h2 = synthetic.spacing2(max(grid))
    s = jb.Solver(grid, blocks, torch.float64, device=device)
    try:
        s.set_state(torch.from_numpy(U).to(device))
        if src:
            s.set_source(torch.from_numpy(f).to(device), h2)
        got = s.residual()
    finally:
        s.close()
    want = oracle.residual(U, oracle.scale_source(f, h2, np.float64) if src else None)
    assert abs(got - want) <= 1e-12 * want


def test_3d_wide_offsets(device):
    """A z layer of blocks of more than 4 GiB (8 x 1 x 690 cells in 32 x 256 narrow
    blocks): the pass runs on 64-bit lane offsets."""
    nx, ny, nz = 256, 256, 690
    rng = np.random.default_rng(6)
    U0 = rng.uniform(0, 1, (nz + 2, ny + 2, nx + 2))
    f = rng.uniform(-1, 1, (nz, ny, nx))
    check(U0, f, synthetic.spacing2(nz), 5, 4, (32, 256, 1), np.float32, device, "3d wide")


# The explicit-halo sweep sends its edge cells itself where blocks span a wave's
# columns or the work items are few, else an exchange launch follows it.
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("case", [(1024, 1024, 64, 64), (1000, 1030, 63, 61), (513, 300, 2, 3)])
def test_explicit_send_rule(device, dtype, case):
    from paper_2303_02543_amd import JACOBI_FLAG_EXPLICIT_HALO
    nx, ny, bx, by = case
    U0 = RNG.uniform(0, 1, (ny + 2, nx + 2))
    f = RNG.uniform(-1, 1, (ny, nx))
    for src in (f, None):
        check(U0, src, synthetic.spacing2(max(nx, ny)), 7, 3, (bx, by), dtype, device,
              "explicit %s" % (case,), depth=1, flags=JACOBI_FLAG_EXPLICIT_HALO)


# Faces of up to 4, 8, ... 128 cells share workgroups, longer ones do not;
# narrow and tall blocks, flat ones, and 3D faces of unequal size.  x blocks of
# 32 columns or fewer: no sweep sends its cells itself.
FACES = [
    # (grid, blocks)
    ((131, 60), (17, 5)),
    ((600, 203), (15, 7)),
    ((2000, 1300), (50, 26)),
    ((1900, 900), (15, 7)),
    ((512, 2611), (64, 2)),
    ((16, 70000), (2, 240)),
    ((40, 33, 29), (5, 4, 6)),
    ((24, 10, 11), (3, 4, 3)),
    ((96, 20, 70), (3, 2, 7)),
    ((70, 41, 130), (2, 2, 3)),
    ((33, 300, 9), (2, 3, 3)),
]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("case", FACES)
def test_face_exchange_and_sends(device, dtype, case):
    from paper_2303_02543_amd import JACOBI_FLAG_EXPLICIT_HALO, JACOBI_FLAG_OVERLAP
    grid, blocks = case
    shape = tuple(reversed(grid))
    U0 = RNG.uniform(0, 1, tuple(n + 2 for n in shape))
    f = RNG.uniform(-1, 1, shape)
    # rows 1: 2D sweeps that leave the exchange to its own launch
    for flags, rows in ((JACOBI_FLAG_EXPLICIT_HALO, 1 if len(grid) == 2 else 0),
                        (JACOBI_FLAG_EXPLICIT_HALO | JACOBI_FLAG_OVERLAP, 0)):
        check(U0, f, synthetic.spacing2(max(grid)), 6, 4, blocks, dtype, device,
              "faces %s %s flags %d" % (case, np.dtype(dtype).name, flags), depth=1, rows=rows,
              flags=flags)


# Tiles of 64 rows, two rows per lane (grids that fill the GPU with them), whose
# last group ends just before, at and just beyond the ring: at depth 5 k groups
# cover 56 k + 8 rows, and an odd number of rows ends inside a lane's pair.
TILES_3D_64 = [
    # (nx, ny, nz, bx, by, bz)
    (513, 232, 160, 5, 4, 2),
    (514, 233, 150, 3, 5, 3),
    (511, 231, 155, 4, 3, 2),
]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("case", TILES_3D_64)
def test_3d_tall_tile_edges(device, dtype, case):
    nx, ny, nz, bx, by, bz = case
    rng = np.random.default_rng(8)
    U0 = rng.uniform(0, 1, (nz + 2, ny + 2, nx + 2))
    f = rng.uniform(-1, 1, (nz, ny, nx))
    h2 = synthetic.spacing2(nx)
    for src, K, R in ((f, 10, 5), (None, 6, 3)):
        check(U0, src, h2, K, R, (bx, by, bz), dtype, device,
              "3d tall tiles %s %s K %d" % (case, np.dtype(dtype).name, K))


# FP32 passes on the row kernel: depth 1 of plates and from 1.05e8 cells on, depths
# 2 - 4 from 2^26 cells on where its rounds are the shorter ones.
ROWS_3D_F32 = [
    # (nx, ny, nz, bx, by, bz, depth)
    (1025, 1021, 3, 4, 3, 1, 1),
    (480, 500, 441, 5, 4, 5, 1),
    (419, 401, 403, 3, 4, 5, 2),
    (419, 401, 403, 4, 3, 2, 3),
    (2000, 600, 60, 9, 4, 2, 4),
]


@pytest.mark.parametrize("case", ROWS_3D_F32)
def test_3d_rows_fp32(device, case):
    nx, ny, nz, bx, by, bz, depth = case
    rng = np.random.default_rng(9)
    U0 = rng.uniform(0, 1, (nz + 2, ny + 2, nx + 2))
    f = rng.uniform(-1, 1, (nz, ny, nx))
    h2 = synthetic.spacing2(max(nx, ny, nz))
    for src in (f, None):
        check(U0, src, h2, depth + 1, depth, (bx, by, bz), np.float32, device,
              "3d rows fp32 %s %s" % (case, "laplace" if src is None else "poisson"), depth=depth)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("case", [(256, 256, 256, 4, 4, 4), (512, 127, 256, 6, 2, 3),
                                  (512, 256, 255, 8, 3, 4)])
def test_3d_rows_whole_rounds(device, dtype, case):
    """Single sweeps of grids that row tiles cover in one round of one or two
    workgroups per CU, exactly and one row or plane short."""
    nx, ny, nz, bx, by, bz = case
    U0 = RNG.uniform(0, 1, (nz + 2, ny + 2, nx + 2))
    f = RNG.uniform(-1, 1, (nz, ny, nx))
    for src in (f, None):
        check(U0, src, synthetic.spacing2(nx), 3, 2, (bx, by, bz), dtype, device,
              "3d whole rounds %s %s source %s" % (case, np.dtype(dtype).name, src is not None), depth=1)


def test_3d_plates_of_double_precision(device):
    """Plates run four sweeps per pass in FP64 (the launches are counted), with
    the result of any other schedule."""
    import torch
    import paper_2303_02543_amd as jb
    nx, ny, nz = 1024, 1023, 3
    rng = np.random.default_rng(10)
    U0 = rng.uniform(0, 1, (nz + 2, ny + 2, nx + 2))
    f = rng.uniform(-1, 1, (nz, ny, nx))
    check(U0, f, synthetic.spacing2(nx), 9, 8, (4, 3, 1), np.float64, device, "plate")
    s = jb.Solver((nx, ny, nz), (4, 3, 1), torch.float64, device=device)
    try:
        s.set_state(torch.zeros(s.state_shape, dtype=torch.float64, device=device))
        s.profile(True)
        s.sweep(20)
        assert s.profile_read(4)["launches"] == 5
        s.profile(False)
    finally:
        s.close()


# Block layouts whose planes share workgroups (few rows of few cells: the last
# group of planes full, short by one, or one plane alone), and such as leave one
# piece per thread or several: into the blocks, explicit sweeps that
# read the frames, and back out.
LAYOUTS = [
    # (grid, blocks)
    ((40, 40, 40), (5, 5, 5)),
    ((39, 33, 31), (3, 4, 2)),
    ((8, 9, 130), (1, 1, 9)),
    ((64, 30, 14), (1, 2, 1)),
    ((16, 8, 6), (2, 1, 1)),
    ((130, 70, 15), (2, 1, 1)),
    ((3000, 40), (4, 3)),
    ((1100, 1030), (2, 2)),
]


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("case", LAYOUTS)
def test_block_layouts(device, dtype, case):
    import torch
    import paper_2303_02543_amd as jb
    grid, blocks = case
    shape = tuple(reversed(grid))
    U0 = RNG.uniform(0, 1, tuple(n + 2 for n in shape)).astype(dtype)
    f = RNG.uniform(-1, 1, shape).astype(dtype)
    h2 = synthetic.spacing2(max(grid))
    s = jb.Solver(grid, blocks, getattr(torch, np.dtype(dtype).name), device=device)
    try:
        s.set_source(torch.from_numpy(f).to(device), h2)
        s.set_state(torch.from_numpy(U0).to(device))
        assert bits_equal(s.get_state().cpu().numpy(), U0), case
    finally:
        s.close()
    check(U0, f, h2, 2, 1, blocks, dtype, device, "layout %s %s" % (case, np.dtype(dtype).name),
          depth=1, flags=jb.JACOBI_FLAG_EXPLICIT_HALO)


def test_small_blocks_keep_the_lanes_busy(device):
    """A source of 256^3 into blocks of 8^3 cells takes about twice as long as into
    64^3 (48 and 22 us); with a plane of 16 lanes per workgroup it took 12 times."""
    import torch
    import paper_2303_02543_amd as jb

    def source_ms(nb):
        s = jb.Solver((256,) * 3, (nb,) * 3, torch.float32, device=device)
        try:
            f = torch.zeros(s.interior_shape, dtype=torch.float32, device=device)
            best = 1e9
            for _ in range(6):
                a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                a.record()
                for _ in range(10):
                    s.set_source(f, 1e-6)
                b.record()
                b.synchronize()
                best = min(best, a.elapsed_time(b))
            return best / 10
        finally:
            s.close()

    small, large = source_ms(32), source_ms(4)
    say("source into blocks", small, large)
    assert small < 6 * large


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("case", [(65, 33, 2, 3, 8), (300, 201, 2, 2, 13), (1000, 777, 4, 3, 13),
                                  (2049, 1030, 8, 8, 16)])
def test_2d_register_tiles_nontemporal(device, dtype, case):
    """The outputs of register tiles stored with the non-temporal hint."""
    from paper_2303_02543_amd import JACOBI_FLAG_NT_STORES
    nx, ny, bx, by, t = case
    U0 = RNG.uniform(0, 1, (ny + 2, nx + 2))
    f = RNG.standard_normal((ny, nx)) * 100
    check(U0, f, synthetic.spacing2(max(nx, ny)), 2 * t + 1, t, (bx, by), dtype, device,
          "2d tiles nt %s %s" % (case, np.dtype(dtype).name), flags=JACOBI_FLAG_NT_STORES)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("case", [((203, 150), (3, 4), 0), ((1200, 1100), (4, 4), 0),
                                  ((70, 41, 33), (2, 2, 3), 5), ((256, 255, 257), (4, 3, 2), 4),
                                  ((419, 401, 203), (4, 3, 2), 2)])
def test_poisoned_workspace_default_schedule(device, dtype, case):
    """A workspace full of NaN under the schedules that the library picks: register
    tiles in 2D, tiles or rows in 3D."""
    import torch
    import paper_2303_02543_amd as jb
    grid, blocks, depth = case
    shape = tuple(reversed(grid))
    tdt = getattr(torch, np.dtype(dtype).name)
    U0 = RNG.uniform(0, 1, tuple(n + 2 for n in shape))
    f = RNG.uniform(-1, 1, shape)
    h2 = synthetic.spacing2(max(grid))
    want, _ = oracle_run(U0, f, h2, 9, dtype)
    s = jb.Solver(grid, blocks, tdt, device=device)
    try:
        s.workspace.view(torch.int32).fill_(-1)  # NaN in either type
        s.set_tuning(depth, 0, 0)
        s.set_state(torch.from_numpy(U0.astype(dtype)).to(device))
        s.set_source(torch.from_numpy(f.astype(dtype)).to(device), h2)
        s.sweep(9)
        assert bits_equal(s.get_state().cpu().numpy(), want), case
        assert np.isfinite(s.residual())
    finally:
        s.close()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("case", [((203, 150), (3, 4), 0), ((1200, 1100), (4, 4), 0),
                                  ((70, 41, 33), (2, 2, 3), 0), ((256, 130, 257), (4, 3, 2), 0),
                                  ((203, 150), (3, 4), 4), ((70, 41, 33), (2, 2, 3), 2)])
def test_one_handle_through_every_schedule(device, dtype, case):
    """Fused passes, explicit exchanges and overlapped sends in turn on one handle
    (deep halos too): each finds the halos that it reads in order."""
    import torch
    import paper_2303_02543_amd as jb
    grid, blocks, halo = case
    shape = tuple(reversed(grid))
    tdt = getattr(torch, np.dtype(dtype).name)
    U0 = RNG.uniform(0, 1, tuple(n + 2 for n in shape))
    f = RNG.uniform(-1, 1, shape)
    h2 = synthetic.spacing2(max(grid))
    explicit = jb.JACOBI_FLAG_EXPLICIT_HALO
    turns = [(0, 5), (explicit, 3), (0, 4), (explicit | jb.JACOBI_FLAG_OVERLAP, 3), (0, 1),
             (explicit, 1), (explicit | jb.JACOBI_FLAG_OVERLAP, 1), (explicit, 2), (0, 6)]
    if halo:
        turns = [(fl, k) for fl, k in turns if not fl & jb.JACOBI_FLAG_OVERLAP]
    want = np.asarray(U0, dtype=dtype)
    b = oracle.scale_source(f.astype(dtype), h2, dtype)
    s = jb.Solver(grid, blocks, tdt, device=device, halo=halo)
    try:
        s.set_state(torch.from_numpy(want).to(device))
        s.set_source(torch.from_numpy(f.astype(dtype)).to(device), h2)
        for flags, k in turns:
            s.set_tuning(0, 0, flags)
            s.sweep(k)
            want = oracle.sweep(want, b, k)
            assert bits_equal(s.get_state().cpu().numpy(), want), (case, flags, k)
    finally:
        s.close()


def test_3d_wide_offsets_double_precision(device):
    """The z layer of more than 4 GiB in FP64."""
    nx, ny, nz = 256, 256, 345
    rng = np.random.default_rng(16)
    U0 = rng.uniform(0, 1, (nz + 2, ny + 2, nx + 2))
    f = rng.uniform(-1, 1, (nz, ny, nx))
    check(U0, f, synthetic.spacing2(nz), 5, 4, (32, 256, 1), np.float64, device, "3d wide FP64")
