"""usp_densify into destinations that take 16-byte stores and into those that do not (odd K, odd row
stride, a base 2 bytes off), bit for bit; nothing outside the matrix is written."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,ld_extra,offset", [(33, 512, 0, 0), (33, 520, 8, 0), (17, 264, 3, 0), (33, 512, 0, 1),
                                                 (33, 509, 3, 0), (1, 8, 0, 0), (16, 7, 1, 0)])
def test_destinations(M, K, ld_extra, offset):
    import torch
    from paper_2607_08786_amd import usp
    W, mask, _ = wl.make_random(M, K, 1, 0.5, seed=M + K)
    A = usp.SparseMatrix(W, mask)
    ld = K + ld_extra
    buf = torch.full((M * ld + offset + 8,), 7.0, dtype=torch.float16, device="cuda")
    out = buf[offset:offset + M * ld].view(M, ld)
    usp.usp_densify(A.handle, out[:, :K])
    torch.cuda.synchronize()
    A.free()
    got = out.cpu().numpy().view(np.uint16)
    assert np.array_equal(got[:, :K], np.where(mask != 0, W, 0))
    seven = np.float16(7.0).view(np.uint16)
    assert (got[:, K:] == seven).all()
    assert (buf[:offset] == 7).all().item() and (buf[offset + M * ld:] == 7).all().item()
