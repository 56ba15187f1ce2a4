"""The fused epilogue's code must not cost a kernel the wavefronts it runs on: the direct-to-LDS kernel keeps
seven wavefronts per CU at two token blocks (two per SIMD), which the planner's grid shows, and a call without
an epilogue gives the values of one whose epilogue changes nothing."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,plan", [
    (28672, 8192, 32, "dma nb=2 tg=1 grid=1792"),
    (28672, 8192, 16, "dma nb=1 tg=1 grid=1792"),
    (5120, 5120, 128, "share nb=2 grid=256 pipelined"),
    (13824, 5120, 150, "share nb=3 grid=256 pipelined"),
    (5120, 5120, 16, "chunk S=5 W=8 nb=1 grid=200"),
    (13824, 5120, 32, "fourwave passes=1 nt=2 grid=512"),
])
def test_grid_and_bits(M, K, N, plan):
    import torch
    from paper_2607_08786_amd import usp
    W, mask, X = wl.make_random(M, K, N, 0.5, seed=M + N)
    A = usp.SparseMatrix(W, mask)
    print(f"case M={M} K={K} N={N}: {A.plan(N)}", flush=True)
    assert A.plan(N) == plan
    Xd = torch.from_numpy(X.view(np.float16)).cuda()
    plain = A.spmm(Xd)
    zero = torch.zeros(M, dtype=torch.float16, device="cuda")
    added = A.spmm(Xd, bias=zero)
    torch.cuda.synchronize()
    A.free()
    assert torch.isfinite(plain).all()
    assert torch.equal(plain, added)  # by value: -0 + 0 is 0
