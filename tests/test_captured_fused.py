"""The benchmark's path, strategy C captured in graphs (mode fused+graph), with
replays: bit for bit against the CPU oracle on small grids, and at the
benchmark's sizes against the undivided grid by several sweeps per launch,
which the full-run oracle tests check."""
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NTH = min(16, os.cpu_count() or 1)
BC = (0.25, -0.5, 1.0, 0.0, -0.75, 0.5)


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import oracle
    from paper_2202_11819_amd import api
    oracle.lib()
    return oracle, api


@pytest.mark.parametrize("n, nblk, split", [
    ((64, 64, 64), (1, 1, 1), None), ((96, 64, 80), (3, 4, 2), None),
    ((75, 60, 41), (2, 3, 3), ([30, 45], [19, 20, 21], [1, 20, 20]))])
def test_replays_match_oracle(env, n, nblk, split):
    # two, three and one replays of 50 sweeps, an odd count of single sweeps
    # behind each (so the next graph starts from the other buffer), other modes
    # and a reload in between
    oracle, api = env
    done = 0
    with api.Solver(n, nblk=nblk, split=split, bc=BC, seed=4) as s:
        for k, mode in ((103, "fused+graph"), (1, "fused"), (157, "fused+graph"), (6, "graph"), (51, "fused+graph"),
                        (100, "fused+graph")):
            print(f"case {n} as {nblk}: {k} sweeps {mode} after {done}", flush=True)
            r = s.run(k, mode=mode, residual=True)
            done += k
            want, want_r, _ = oracle.jacobi(n, done, bc=BC, seed=4, nthreads=NTH)
            assert np.array_equal(s.get_interior(), want) and r == want_r, (mode, done)
        s.set_interior(want)
        assert s.run(101, mode="fused+graph", residual=True) > 0
        want, _, _ = oracle.jacobi(n, done + 101, bc=BC, seed=4, nthreads=NTH)
        assert np.array_equal(s.get_interior(), want)


def _undivided(api, n, seed, sweeps):
    with api.Solver(n, seed=seed) as s:
        r = s.run(sweeps, mode="graph", residual=True)
        return s.get_interior_device(), r


def test_benchmark_step_512(env):
    # 512^3 as 8^3 blocks, 1000 sweeps: 19 replays, then 50 single sweeps
    import torch
    _, api = env
    n = (512, 512, 512)
    want, want_r = _undivided(api, n, 1, 1000)
    with api.Solver(n, nblk=(8, 8, 8), seed=1) as s:
        r = s.run(1000, mode="fused+graph", residual=True)
        assert r == want_r
        assert torch.equal(s.get_interior_device().view(torch.int64), want.view(torch.int64))


def test_decompositions_1024(env):
    import torch
    _, api = env
    from paper_2202_11819_amd import workloads as W
    want = None
    for label, spec in W.block_sweep():
        print(label, flush=True)
        if want is None:
            want, want_r = _undivided(api, spec.n, spec.seed, 101)
        with api.Solver(spec.n, nblk=spec.nblk, split=spec.split, seed=spec.seed) as s:
            assert s.run(101, mode="fused+graph", residual=True) == want_r, label
            got = s.get_interior_device()
        assert torch.equal(got.view(torch.int64), want.view(torch.int64)), label
        del got
