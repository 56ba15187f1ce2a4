"""The fused epilogue's operands read as 8-byte vectors or one value at a time: a bias 2 bytes off an
8-byte boundary and a residual whose rows start at any alignment give the same bits as aligned ones,
in every kernel, on row blocks that are split and on those that are not."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N,act,route", [
    (1024, 1024, 16, "silu", "row"),
    (4101, 1000, 16, "relu", "chunk S=1"),
    (4101, 3000, 16, "gelu_tanh", "chunk S=3"),
    (5120, 5120, 30, "gelu_tanh", "chunk S=5 W=8 nb=2"),
    (1100, 1000, 20, "silu", "fourwave"),
    (4101, 1000, 48, "none", "fourwave"),
    (36880, 8088, 16, "relu", "dma"),
    (13824, 5120, 64, "silu", "share nb=1"),
    (5120, 5120, 100, "gelu_tanh", "share nb=2"),
    (8200, 2000, 200, "relu", "wide passes=1 nb=1"),
    (1101, 700, 333, "silu", "wide"),
])
def test_same_bits(M, K, N, act, route):
    import torch
    from paper_2607_08786_amd import usp
    W, mask, X = wl.make_random(M, K, N, 0.5, seed=M + N)
    A = usp.SparseMatrix(W, mask)
    plan = A.plan(N)
    print(f"case M={M} K={K} N={N}: {plan}", flush=True)
    assert plan.startswith(route), plan
    g = torch.Generator(device="cuda").manual_seed(3)
    Xd = torch.from_numpy(X.view(np.float16)).cuda()
    ld = (M + 7) // 8 * 8
    bias = torch.randn(ld, generator=g, device="cuda", dtype=torch.float16)[:M]
    res = torch.randn(N, ld, generator=g, device="cuda", dtype=torch.float16)[:, :M]
    bias1 = torch.cat([bias[:1], bias])[1:]
    res1 = torch.empty(N * (ld + 1) + 1, device="cuda", dtype=torch.float16)[1:].view(N, ld + 1)[:, :M]
    res1.copy_(res)
    assert bias.data_ptr() % 8 == 0 and bias1.data_ptr() % 8 == 2 and res1.data_ptr() % 8 == 2
    want = A.spmm(Xd, bias=bias, residual=res, activation=act)
    got = A.spmm(Xd, bias=bias1, residual=res1, activation=act)
    only = A.spmm(Xd, bias=bias1, activation=act)
    ref = A.spmm(Xd, bias=bias, activation=act)
    torch.cuda.synchronize()
    A.free()
    assert torch.isfinite(want).all()
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    assert torch.equal(only.view(torch.int16), ref.view(torch.int16))
