"""Several sweeps per launch (GRAPH, TWO_SWEEP, batches, pools, the one-shot
solve): the tile tables on the host, and on the GPU the bits of the CPU oracle
(tolerance zero: the same operations in the same order)."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NTH = min(16, os.cpu_count() or 1)
BC = (0.25, -0.5, 1.0, 0.0, -0.75, 0.5)


def test_tiles_cover_every_cell_and_fit_their_shape(tmp_path):
    pkg = os.path.join(ROOT, "paper_2202_11819_amd")
    exe = tmp_path / "multi_tile_check"
    src = os.path.join(ROOT, "tests", "multi_tile_check.cpp")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(pkg, "csrc"), "-I", os.path.join(ROOT, "include"), src,
                           "-o", str(exe), "-L", pkg, "-lj3d", f"-Wl,-rpath,{pkg}"])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout[-2000:]
    assert " 0 bad" in out.stdout


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import oracle
    from paper_2202_11819_amd import api, j3d
    oracle.lib()
    return oracle, api, j3d


# undivided: one lane wide, the widest single tile and one cell more, tiles cut
# along every axis, one plane; even blocks: one cell thick, thinner than a
# launch's sweeps, tiles across several blocks; uneven blocks: rows that end
# inside tiles, as shallow as the planner takes and too shallow for it
GRIDS = [((1, 1, 1), (1, 1, 1), None), ((62, 30, 9), (1, 1, 1), None), ((63, 31, 40), (1, 1, 1), None),
         ((130, 70, 37), (1, 1, 1), None), ((241, 3, 4), (1, 1, 1), None), ((2, 150, 1), (1, 1, 1), None),
         ((200, 300, 260), (1, 1, 1), None),
         ((5, 4, 3), (5, 4, 3), None), ((96, 64, 80), (3, 4, 2), None), ((128, 96, 30), (4, 4, 15), None),
         ((320, 256, 256), (5, 4, 4), None),
         ((37, 29, 23), (3, 2, 4), ([10, 20, 7], [1, 28], [5, 5, 6, 7])),
         ((150, 170, 133), (2, 3, 3), ([60, 90], [50, 57, 63], [40, 50, 43])),
         ((130, 40, 12), (2, 1, 3), ([1, 129], None, [3, 2, 7])),
         ((300, 260, 250), (3, 2, 2), ([64, 130, 106], [100, 160], [121, 129]))]


@pytest.mark.gpu
@pytest.mark.parametrize("n, nblk, split", GRIDS)
def test_every_count_matches_oracle(env, n, nblk, split):
    # counts below, at and past one launch's sweeps; the residual of the last sweep
    oracle, api, _ = env
    for iters in (1, 4, 11):
        print(f"case {n} as {nblk}, {iters} sweeps", flush=True)
        want, want_r, _ = oracle.jacobi(n, iters, bc=BC, seed=6, nthreads=NTH)
        with api.Solver(n, nblk=nblk, split=split, bc=BC, seed=6) as s:
            assert s.run(iters, mode="graph", residual=True) == want_r
            assert np.array_equal(s.get_interior(), want), (n, nblk, iters)


@pytest.mark.gpu
def test_faces_modes_and_replays(env):
    # per-cell boundary values; runs without a residual, graph replays with eager
    # work between them, the one-sweep modes in between (their halos are stale
    # after a multi-sweep run and fetched again), an explicit shape at the end
    oracle, api, _ = env
    n, nblk = (77, 60, 64), (1, 3, 2)
    rng = np.random.default_rng(5)
    nx, ny, nz = n
    faces = [rng.uniform(-1, 1, s) for s in [(nz, ny), (nz, ny), (nz, nx), (nz, nx), (ny, nx), (ny, nx)]]
    plan = [(5, "fused"), (203, "graph"), (3, "fused"), (2, "unfused_phase"), (130, "graph"), (7, "block_c"),
            (121, "graph"), (3, "fused+graph")]
    done = 0
    with api.Solver(n, nblk=nblk, seed=8) as s:
        for f in range(6):
            s.set_face(f, faces[f])
        for k, mode in plan:
            print(f"{k} sweeps {mode}", flush=True)
            r = s.run(k, mode=mode, residual=done % 2 == 0)
            done += k
            want, want_r, _ = oracle.jacobi(n, done, seed=8, faces=faces, nthreads=NTH)
            assert np.array_equal(s.get_interior(), want), (mode, done)
            assert r is None or r == want_r
        s.set_tune(25, 16, 0)  # the caller's one-sweep shape
        r = s.run(60, mode="graph", residual=True)
        want, want_r, _ = oracle.jacobi(n, done + 60, seed=8, faces=faces, nthreads=NTH)
        assert np.array_equal(s.get_interior(), want) and r == want_r


@pytest.mark.gpu
@pytest.mark.parametrize("two", [False, True])
def test_batch_of_decomposed_and_undivided_problems(env, two):
    # counts 0 and around multiples of a launch's sweeps; uneven blocks put the
    # whole batch on the general kernel
    oracle, api, j3d = env
    specs = [((40, 33, 27), (1, 1, 1), None, 0), ((64, 64, 64), (1, 1, 1), None, 13), ((7, 90, 31), (1, 1, 1), None, 3),
             ((100, 37, 50), (1, 1, 1), None, 16)]
    if not two:
        specs += [((96, 48, 40), (3, 2, 2), None, 9), ((60, 50, 45), (2, 1, 2), ([17, 43], None, [21, 24]), 30)]
    probs = [j3d.Problem(n, b, sp, BC, 9, i) for i, (n, b, sp, _) in enumerate(specs)]
    with api.Batch(probs, [it for *_, it in specs]) as batch:
        res = batch.run(two_sweep=two)
        for i, (n, _, _, it) in enumerate(specs):
            want, want_r, _ = oracle.jacobi(n, it, bc=BC, seed=9, pid=i, nthreads=NTH)
            assert np.array_equal(batch.get_interior(i), want) and res[i] == want_r, i


@pytest.mark.gpu
def test_noalloc_counts_and_decompositions(env):
    import torch
    oracle, _, j3d = env
    for n, nblk, split, iters in [((48, 40, 36), (3, 2, 3), None, 23), ((66, 31, 25), (1, 1, 1), None, 1),
                                  ((90, 64, 50), (2, 1, 2), ([30, 60], None, [20, 30]), 14)]:
        p = j3d.Problem(n, nblk, split, BC, 7, 0)
        nbytes = j3d.j3d_field_bytes(p)
        fields = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        out = torch.empty(n[::-1], dtype=torch.float64, device="cuda")
        r = j3d.j3d_solve_noalloc(p, fields.data_ptr(), nbytes, None, out.data_ptr(), iters, True,
                                  torch.cuda.current_stream().cuda_stream)
        want, want_r, _ = oracle.jacobi(n, iters, bc=BC, seed=7, nthreads=NTH)
        assert np.array_equal(out.cpu().numpy(), want) and r == want_r, (n, nblk)


@pytest.mark.gpu
@pytest.mark.parametrize("n, nblk, split", [
    ((64, 32, 6), (1, 1, 1), None), ((63, 33, 5), (1, 1, 1), None),       # one run, and one cell past it
    ((128, 64, 40), (4, 2, 5), None), ((126, 22, 9), (3, 2, 3), None),    # pairs; planes below half a run
    ((30, 28, 20), (3, 4, 2), ([9, 11, 10], [7, 7, 7, 7], [1, 19])),      # odd rows inside an even grid
    ((5, 4, 3), (5, 4, 3), None), ((1, 1, 1), (1, 1, 1), None), ((2, 2100, 3), (1, 1, 1), None)])
def test_interior_copies_both_ways(env, n, nblk, split):
    # device arrays on 16 bytes and 8 bytes past them, host arrays
    import torch
    _, api, j3d = env
    count = n[0] * n[1] * n[2]
    u = torch.rand(count + 1, dtype=torch.float64, device="cuda")
    with api.Solver(n, nblk=nblk, split=split) as s:
        for at in (0, 1):
            src = u[at:at + count]
            out = torch.full((count + 1,), -1.0, dtype=torch.float64, device="cuda")
            j3d.j3d_set_interior(s.h, src.data_ptr(), True)
            j3d.j3d_get_interior(s.h, out[1 - at:].data_ptr(), True)
            torch.cuda.synchronize()
            assert torch.equal(out[1 - at:1 - at + count], src)
            assert out[0 if at == 0 else count] == -1.0  # nothing written past either end
            assert np.array_equal(s.get_interior().ravel(), src.cpu().numpy())
            s.set_interior(src.cpu().numpy()[::-1])
            assert np.array_equal(s.get_interior().ravel(), src.cpu().numpy()[::-1])
