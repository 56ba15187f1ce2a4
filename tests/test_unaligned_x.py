"""GPU parity where X is not 16-byte aligned or K and ldx are no multiples of 8,
through the C ABI: every kernel that takes such calls, exact on small integers.
One token is all Inf and one all NaN: the chunk of columns that straddles K must
not bring another token's values into a product (0 x Inf is NaN)."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu


# K mod 8 from 1 to 7 and 0; rows of X that start at every alignment (ldx odd or
# even, the base 2 bytes off or not).
@pytest.mark.parametrize("M,K,N,ldx_extra,offset,route", [
    (1025, 1021, 7, 0, 0, "fourwave"),           # one chunk of columns
    (1025, 1, 3, 0, 1, "fourwave"),
    (3583, 8191, 8, 0, 1, "chunk S=8 W=8 nb=1"),
    (8191, 2045, 16, 0, 0, "fourwave"),          # few tiles and chunks
    (4999, 4093, 4, 0, 1, "fourwave"),           # more of them: up to 4 tokens
    (4999, 4093, 5, 0, 1, "chunk S=4 W=8 nb=1"),
    (13821, 5117, 3, 0, 0, "fourwave"),          # several rounds of workgroups
    (4999, 4093, 21, 0, 0, "chunk S=4 W=8 nb=2"),
    (13821, 5117, 16, 3, 1, "chunk S=5 W=4 nb=1"),
    (5120, 5120, 16, 3, 1, "chunk S=5 W=8 nb=1"),
    (5120, 5120, 30, 4, 1, "chunk S=5 W=8 nb=2"),
    (1024, 1024, 16, 8, 1, "row"),               # aligned calls take the row kernel, this one the passes
    (4101, 1001, 48, 0, 0, "fourwave"),
    (4101, 1006, 200, 1, 0, "fourwave"),
    (36880, 8083, 16, 0, 0, "dma nb=1"),         # X copied to padded rows
    (36880, 8082, 27, 0, 1, "dma nb=2"),
    (36880, 8088, 20, 1, 0, "dma nb=2"),         # K a multiple of 8: the passes
    (13824, 5115, 60, 0, 0, "share nb=1"),
    (28672, 5120, 100, 3, 1, "share nb=2"),
    (5120, 5114, 100, 2, 0, "share nb=2"),       # pipelined
    (36880, 2047, 180, 0, 0, "share nb=3"),
])
def test_exact(M, K, N, ldx_extra, offset, route):
    import torch
    from paper_2607_08786_amd import usp
    W, mask, X = wl.make_small_int(M, K, N, 0.5, seed=M + K + N, lo=-1, hi=1)
    A = usp.SparseMatrix(W, mask)
    plan = A.plan(N)
    print(f"case M={M} K={K} N={N} ldx={K + ldx_extra} offset={offset}: {plan}", flush=True)
    assert plan.startswith(route), plan
    rows = None
    if M * K * N > 2 ** 31:
        rows = np.unique(np.concatenate([np.random.default_rng(1).choice(M, 300, replace=False), [0, M - 1]]))
    Yref, _ = oracle.masked_gemm(W, mask, X, rows=rows)
    Xh = X.view(np.float16).copy()
    Xh[1], Xh[N - 1] = np.inf, np.nan
    ldx = K + ldx_extra
    buf = torch.full((N * ldx + offset,), float("nan"), dtype=torch.float16, device="cuda")
    Xd = buf[offset:].view(N, ldx)[:, :K]
    Xd.copy_(torch.from_numpy(Xh).cuda())
    Y = A.spmm(Xd)
    torch.cuda.synchronize()
    A.free()
    got = Y.cpu().numpy().astype(np.float64)
    got = got if rows is None else got[:, rows]
    plain = [n for n in range(N) if n not in (1, N - 1)]
    assert np.array_equal(got[plain], Yref[plain])
    assert not np.isfinite(got[1][np.abs(Yref[1]) > 0]).any()  # rows with kept weights meet the Inf


# K no multiple of 8 on a layer whose partials leave the device scratch no room for the padded copy of X: no copy
# is made, whether the workspace is the scratch (refused, as before) or a tensor.
def test_no_room_for_the_padded_copy():
    import torch
    from paper_2607_08786_amd import usp
    M, K, N = 131072, 1789, 32
    rng = np.random.default_rng(3)
    W, mask = np.zeros((M, K), dtype=np.uint16), np.zeros((M, K), dtype=np.uint8)
    rows = np.array([0, 5, 70001, M - 1])
    for r in rows:
        W[r] = rng.choice(np.array([-1, 0, 1], dtype=np.float16), K).view(np.uint16)
        mask[r] = rng.random(K) < 0.5
    X = rng.choice(np.array([-1, 0, 1], dtype=np.float16), (N, K))
    A = usp.SparseMatrix(W, mask)
    print(f"case M={M} K={K} N={N}: {A.plan(N)}, workspace {A.workspace_size(N)} bytes", flush=True)
    assert A.plan(N).startswith("fourwave") and A.workspace_size(N) > usp.NOALLOC_SCRATCH_BYTES
    Xd = torch.from_numpy(X).cuda()
    Y = A.spmm(Xd)
    with pytest.raises(usp.UspError) as e:
        usp.usp_spmm_noalloc(A.handle, Xd, torch.empty_like(Y))
    torch.cuda.synchronize()
    A.free()
    assert e.value.status == 2
    got = Y.cpu().numpy().astype(np.float64)
    Yref, _ = oracle.masked_gemm(W, mask, X.view(np.uint16), rows=rows)
    assert np.array_equal(got[:, rows], Yref) and not np.delete(got, rows, axis=1).any()
