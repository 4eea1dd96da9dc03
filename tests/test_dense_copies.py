"""Interior copies between a dense grid and decomposed fields: both forms (by
blocks and by cells, as tests/dense_route_check.cpp lists them), device arrays
on 16 bytes and 8 past them, host arrays in one transfer and in several."""
import numpy as np
import pytest


@pytest.mark.gpu
@pytest.mark.parametrize("n, nblk, split", [
    ((70, 50, 40), (3, 3, 3), ([64, 1, 5], [45, 1, 4], [1, 30, 9])),                 # by cells
    ((152, 128, 254), (3, 2, 5), ([150, 1, 1], [64, 64], [250, 1, 1, 1, 1])),        # by cells, two transfers
    ((152, 256, 150), (2, 2, 2), ([128, 24], [128, 128], [70, 80])),                 # by blocks, two transfers
    ((64, 64, 64), (64, 64, 64), None), ((60, 48, 36), (5, 4, 3), None)])            # single cells; 12^3 blocks
def test_both_forms_copy_every_cell(n, nblk, split):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2202_11819_amd import api, j3d
    print(f"case {n} as {nblk}", flush=True)
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
