"""Every compiled shape of the several-sweeps kernel, its short form (one or two
sweeps) and its remainders, on equal and on unequal blocks, bit for bit against
the CPU oracle (tolerance zero: the same operations in the same order)."""
import ctypes
import os

import numpy as np
import pytest

NTH = min(16, os.cpu_count() or 1)
BC = (0.25, -0.5, 1.0, 0.0, -0.75, 0.5)
SHAPES = 7

# ragged undivided, ragged equal blocks across tiles, unequal blocks whose rows
# are as shallow as five sweeps a launch take
GRIDS = [((131, 75, 23), (1, 1, 1), None), ((96, 80, 30), (4, 4, 3), None),
         ((129, 70, 26), (3, 2, 4), ([50, 9, 70], [31, 39], [5, 9, 6, 6]))]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", range(SHAPES))
@pytest.mark.parametrize("n, nblk, split", GRIDS)
def test_every_shape_and_count(shape, n, nblk, split):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import oracle
    from paper_2202_11819_amd import api, j3d
    oracle.lib()
    force = j3d._lib.j3d_check_multi_shape
    force.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.POINTER(ctypes.c_int32)]
    sweeps = ctypes.c_int32()
    with api.Solver(n, nblk=nblk, split=split, bc=BC, seed=6) as s:
        assert force(s.h, SHAPES, ctypes.byref(sweeps)) == j3d.J3D_EINVAL
        assert force(s.h, shape, ctypes.byref(sweeps)) == j3d.J3D_OK
        t, done = sweeps.value, 0
        for k in (1, 2, t - 1, t, t + 1, t + 2, 2 * t + 1):
            print(f"case {n} as {nblk}, shape {shape}, {k} sweeps after {done}", flush=True)
            r = s.run(k, mode="graph", residual=True)
            done += k
            want, want_r, _ = oracle.jacobi(n, done, bc=BC, seed=6, nthreads=NTH)
            assert np.array_equal(s.get_interior(), want) and r == want_r, (shape, k)
