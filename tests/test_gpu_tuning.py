"""The autotuner and the profiling records, through the C ABI.

Autotuning only picks among schedules that compute identical results, so a
tuned run must still equal the oracle bit for bit; its result is cached per
problem shape in the file JACOBI_TUNE_CACHE names, and a cache line the
library cannot use is ignored (the shape is tuned again).  The profiling
records count exactly the passes the host planner issues: a 25-sweep run at
depth 4 is split into passes of 4, 4, 4, 4, 3, 3, 3 sweeps."""
import sys

import numpy as np
import pytest

import oracle
import synthetic
from gpu_util import bits_equal, to_device

pytestmark = pytest.mark.gpu

RNG = np.random.default_rng(77)


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def _problem(nx, ny):
    U0 = RNG.uniform(0, 1, (ny + 2, nx + 2)).astype(np.float32)
    f = (RNG.standard_normal((ny, nx)) * 100).astype(np.float32)
    return U0, f, synthetic.spacing2(max(nx, ny))


def test_autotune_cache_and_bit_neutral(device, tmp_path, monkeypatch):
    import torch
    import paper_2303_02543_amd as jb
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("JACOBI_TUNE_CACHE", str(cache))
    nx, ny, K = 300, 200, 30
    U0, f, h2 = _problem(nx, ny)
    want = oracle.sweep(U0, oracle.scale_source(f, h2, np.float32), K)
    s1 = jb.Solver((nx, ny), (3, 2), torch.float32, device=device)
    s2 = jb.Solver((nx, ny), (3, 2), torch.float32, device=device)
    try:
        tuned = s1.autotune(10, with_source=True)
        say("autotune ->", tuned)
        lines = cache.read_text().splitlines()
        assert len(lines) == 1 and lines[0].endswith("-> %d %d %d" % tuned)
        # a second handle of the same shape takes the cached schedule
        assert s2.autotune(10, with_source=True) == tuned
        assert len(cache.read_text().splitlines()) == 1
        d2, r2, f2 = s2.get_tuning()
        assert (d2, f2) == (tuned[0], tuned[2]) and (tuned[1] == 0 or r2 == tuned[1])
        s2.set_source(to_device(f, np.float32, device), h2)
        s2.set_state(to_device(U0, np.float32, device))
        s2.sweep(K)
        got = s2.get_state().cpu().numpy()
        assert bits_equal(got, want), "tuned schedule %s" % (tuned,)
        # an unusable cache line (flag bits the library does not know) for
        # this shape is skipped: the shape is tuned again and a line added
        key = lines[0].split(" -> ")[0]
        cache.write_text("%s -> 1 0 1024\n" % key)
        again = s1.autotune(10, with_source=True)
        assert again[0] >= 1 and len(cache.read_text().splitlines()) == 2
    finally:
        s1.close()
        s2.close()


def test_profile_records_count_passes(device):
    import torch
    import paper_2303_02543_amd as jb
    nx, ny, K = 513, 260, 25
    U0, f, h2 = _problem(nx, ny)
    cells = nx * ny
    s = jb.Solver((nx, ny), (3, 5), torch.float32, device=device)
    try:
        s.set_source(to_device(f, np.float32, device), h2)
        s.set_state(to_device(U0, np.float32, device))
        s.set_tuning(4, 0, 0)
        s.profile(True)
        s.sweep(K)
        p = s.profile_read(0)
        p4, p3 = s.profile_read(4), s.profile_read(3)
        s.profile(False)
        say("profile", p, p4, p3)
        assert p["launches"] == 7 and p4["launches"] == 4 and p3["launches"] == 3
        assert p["cell_updates"] == cells * K
        assert p["alg_bytes"] == 7 * cells * 4 * 3  # state r+w, source r, FP32
        assert p["ms"] > 0 and p["ms"] == pytest.approx(p4["ms"] + p3["ms"])
        # the explicit-halo schedule records one launch per sweep
        s.set_tuning(1, 0, jb.JACOBI_FLAG_EXPLICIT_HALO)
        s.profile(True)
        s.sweep(5)
        q = s.profile_read(0)
        s.profile(False)
        assert q["launches"] == 5 and q["cell_updates"] == cells * 5
        got = s.get_state().cpu().numpy()
    finally:
        s.close()
    assert bits_equal(got, oracle.sweep(U0, oracle.scale_source(f, h2, np.float32), K + 5))


@pytest.mark.parametrize("case", [((513, 260), (3, 5), "float32"), ((300, 201), (2, 2), "float64"),
                                  ((2500, 1701), (5, 4), "float64"), ((40, 36, 30), (2, 2, 2), "float32"),
                                  ((96, 96, 96), (2, 2, 2), "float64")])
def test_tuning_read_back_gives_the_schedule_again(device, case):
    """What get_tuning reports is accepted by set_tuning and leaves the passes
    as they were: the launches of a run, counted per depth, stay the same."""
    import torch
    import paper_2303_02543_amd as jb
    grid, blocks, name = case
    s = jb.Solver(grid, blocks, getattr(torch, name), device=device)
    try:
        s.set_state(torch.zeros(s.state_shape, dtype=s.torch_dtype, device=device))
        seen = []
        for _ in range(2):
            counts = []
            for K in (48, 7):
                s.profile(True)
                s.sweep(K)
                counts.append([s.profile_read(d)["launches"] for d in range(1, 17)])
                s.profile(False)
            seen.append(counts)
            t = s.get_tuning()
            say("read back", case, t)
            s.set_tuning(*t)
            assert s.get_tuning() == t
        assert seen[0] == seen[1]
    finally:
        s.close()


@pytest.mark.parametrize("case", [((20000, 500), (20, 1), True, True), ((6000, 2000), (12, 4), True, True),
                                  ((6000, 2000), (12, 4), False, True), ((4096, 2048), (8, 4), False, True),
                                  ((1200, 1100), (4, 4), True, False), ((2500, 2500), (5, 5), True, False)])
def test_2d_single_precision_route(device, case):
    """FP32 grids on which register tiles are slower march for any number of sweeps
    (a tile height is reported; 13 sweeps of 20000x500 with a source 48.6 us, on
    tiles 62.1); smaller ones run on register tiles.  Same states by either."""
    import torch
    import paper_2303_02543_amd as jb
    shape, blocks, src, march = case
    gen = torch.Generator(device).manual_seed(5)
    solvers = [jb.Solver(shape, blocks, torch.float32, device=device) for _ in range(2)]
    try:
        U = torch.rand(solvers[0].state_shape, dtype=torch.float32, device=device, generator=gen)
        f = torch.rand(solvers[0].interior_shape, dtype=torch.float32, device=device, generator=gen)
        for s in solvers:
            if src:
                s.set_source(f, 1e-6)
            s.set_state(U)
        rows = solvers[0].get_tuning()[1]
        say("route", case, rows)
        assert (rows > 0) == march
        solvers[1].set_tuning(5, 16, 0)
        for s in solvers:
            s.sweep(13)
            s.sweep(50)
        assert torch.equal(solvers[0].get_state(), solvers[1].get_state())
    finally:
        for s in solvers:
            s.close()


@pytest.mark.parametrize("case", [((700, 601), (3, 2), "float64"), ((1200, 1000), (4, 4), "float32"),
                                  ((96, 96, 96), (2, 2, 2), "float32")])
def test_autotune_is_not_slower_than_the_default(device, monkeypatch, case):
    """The default schedule is among those the autotuner times, so its pick
    takes at most the default's kernel time (a sixth is left for noise)."""
    import torch
    import paper_2303_02543_amd as jb
    monkeypatch.delenv("JACOBI_TUNE_CACHE", raising=False)
    grid, blocks, name = case
    s = jb.Solver(grid, blocks, getattr(torch, name), device=device)

    def kernel_ms():
        s.set_state(torch.zeros(s.state_shape, dtype=s.torch_dtype, device=device))
        out = []
        for _ in range(7):
            s.profile(True)
            s.sweep(48)
            out.append(s.profile_read(0)["ms"])
            s.profile(False)
        return min(out)

    try:
        default = kernel_ms()
        tuned = s.autotune(48, with_source=False)
        ms = kernel_ms()
        say("autotuned", case, tuned, "%.4f ms, default %.4f" % (ms, default))
        assert ms <= default * 7 / 6
    finally:
        s.close()


def test_tune_cache_lines_of_other_versions_are_not_taken(device, tmp_path, monkeypatch):
    import torch
    import paper_2303_02543_amd as jb
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("JACOBI_TUNE_CACHE", str(cache))
    old = "jacobi-v1 nd=2 n=300,200,1 b=3,2,1 dt=0 src=0 sweeps=20 -> 1 0 1"
    cache.write_text(old + "\n")
    s = jb.Solver((300, 200), (3, 2), torch.float32, device=device)
    try:
        assert s.autotune(20, with_source=False) != (1, 0, 1)
        lines = cache.read_text().splitlines()
        assert lines[0] == old and len(lines) == 2
    finally:
        s.close()
