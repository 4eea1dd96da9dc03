"""Which launches a batch or a pool takes, against the CPU oracle bit for bit:
rounds and batches of very few sweeps, several sweeps asked for in spite of a
one-sweep shape, and a single sweep after several."""
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

NTH = min(16, os.cpu_count() or 1)
BC = (0.25, -0.5, 1.0, 0.0, -0.75, 0.5)
SIZES = [(40, 33, 27), (64, 64, 64), (7, 90, 31), (100, 37, 50), (1, 200, 40)]


@pytest.fixture(scope="module")
def env():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import oracle
    from paper_2202_11819_amd import api, j3d
    oracle.lib()
    return oracle, api, j3d


@pytest.mark.parametrize("two, tune", [(False, None), (True, None), (True, (25, 16)), (False, (25, 16))])
def test_pool_rounds_of_few_sweeps(env, two, tune):
    # rounds of one, two and three sweeps, alone and mixed with longer ones;
    # (True, shape): several sweeps asked for in spite of a one-sweep shape
    oracle, api, j3d = env
    iters = [1, 2, 3, 23, 40]
    probs = [j3d.Problem(n, bc=BC, seed=9, pid=i) for i, n in enumerate(SIZES)]
    with api.Pool(sum(j3d.j3d_pool_request_bytes(p) for p in probs), max_slots=len(probs)) as pool:
        if tune:
            pool.set_tune(*tune)
        pool.set_two_sweep(two)
        for steps in ((1, 2, 3), (2,), (7, 1)):
            slots = [pool.try_admit(p, it, check_every=10) for p, it in zip(probs, iters)]
            done, at = 0, 0
            while done < len(slots):
                finished, busy = pool.poll()
                done += len(finished)
                if not busy and done < len(slots):
                    pool.step(steps[at % len(steps)])
                    at += 1
            for i, slot in enumerate(slots):
                want, want_r, _ = oracle.jacobi(SIZES[i], iters[i], bc=BC, seed=9, pid=i, nthreads=NTH)
                u, r, it = pool.result(slot)
                assert it == iters[i] and r == want_r and np.array_equal(u, want), (steps, i)
            for slot in slots:
                pool.release(slot)


@pytest.mark.parametrize("tune", [None, (25, 16, 0)])
@pytest.mark.parametrize("two", [False, True])
@pytest.mark.parametrize("most", [1, 2, 3, 9])
def test_batches_of_few_sweeps(env, most, two, tune):
    oracle, api, j3d = env
    iters = [max(0, most - i) for i in range(len(SIZES))]
    probs = [j3d.Problem(n, bc=BC, seed=9, pid=i) for i, n in enumerate(SIZES)]
    with api.Batch(probs, iters, tune=tune) as batch:
        res = batch.run(two_sweep=two)
        for i, n in enumerate(SIZES):
            want, want_r, _ = oracle.jacobi(n, iters[i], bc=BC, seed=9, pid=i, nthreads=NTH)
            assert np.array_equal(batch.get_interior(i), want) and res[i] == want_r, i


def test_tune_names_a_shape_or_not(env):
    # GRAPH keeps to a shape the program named, and to nothing else
    import ctypes
    _, api, j3d = env
    look = j3d._lib.j3d_check_multi_shape
    look.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.POINTER(ctypes.c_int32)]

    def sweeps(s):
        v = ctypes.c_int32()
        assert look(s.h, -1, ctypes.byref(v)) == j3d.J3D_OK
        return v.value

    with api.Solver((64, 64, 64)) as s:
        several = sweeps(s)
        assert several > 1
        default = s.get_tune()
        for tune, want in (((25, 16, 0), 1), ((-1, 0, 0), several), ((-1, 32, 0), 1), ((None,), several),
                           (default, 1), ((), several)):
            s.set_tune(*tune)
            assert sweeps(s) == want, tune
        s.set_tune(None)
        assert s.get_tune() == default
    with api.Pool(1 << 24, max_slots=1) as pool:
        pool.set_tune(25, 16)
        pool.set_tune(None)
        with pytest.raises(j3d.J3DError):
            pool.set_tune(-1, 0)


def test_single_sweeps_between_several(env):
    # a single sweep reads halos that a launch of several leaves stale
    oracle, api, _ = env
    n, done = (90, 64, 50), 0
    with api.Solver(n, nblk=(3, 2, 2), bc=BC, seed=3) as s:
        for k in (1, 9, 1, 1, 2, 1, 30, 1, 3):
            r = s.run(k, residual=True)
            done += k
            want, want_r, _ = oracle.jacobi(n, done, bc=BC, seed=3, nthreads=NTH)
            assert np.array_equal(s.get_interior(), want) and r == want_r, (k, done)
