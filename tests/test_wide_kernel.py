"""GPU parity of the wide kernel (193 to 256 tokens on large layers, 320 and more
on every matrix), through the C ABI. Small integers, so every output is exact
whatever the order of the sums: |sum| stays below 2^11, an exact fp16."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available()
    return t


@pytest.fixture(scope="module")
def usp(torch):
    from paper_2607_08786_amd import usp as mod
    mod.load_library()
    return mod


def to_dev(torch, bits, ldx_extra=0, offset=0):
    t = torch.from_numpy(np.ascontiguousarray(bits).view(np.float16)).cuda()
    if not (ldx_extra or offset):
        return t
    N, K = t.shape
    buf = torch.zeros(N * (K + ldx_extra) + offset, dtype=torch.float16, device="cuda")
    v = buf[offset:offset + N * (K + ldx_extra)].view(N, K + ldx_extra)[:, :K]
    v.copy_(t)
    return v


# One token past the lower limit and the limit itself; ragged rows (a set with
# one row), columns (a partial tile, K odd) and tokens; one tile and one unit;
# tiles split evenly over workgroups (one partial slot each) and ranges that
# cross tiles (256 workgroups, two slots); two passes; X unaligned; every record
# size the kernel is built for, and nearly dense records, which it leaves to the
# passes of the four-wavefront kernel.
@pytest.mark.parametrize("M,K,N,density,route,unaligned", [
    (128, 256, 320, 0.5, "wide passes=1", False),
    (1, 1, 321, 1.0, "wide passes=1", True),
    (129, 300, 512, 0.5, "wide passes=1", False),
    (1100, 700, 515, 0.5, "wide passes=1", False),
    (1100, 701, 333, 0.5, "wide passes=1", True),
    (13824, 5120, 640, 0.5, "wide passes=1 nb=1 grid=256", False),
    (200, 500, 2100, 0.5, "wide passes=2", False),
    (300, 1000, 700, 0.02, "wide", False),
    (300, 1000, 700, 0.3, "wide", True),
    (300, 1000, 700, 0.62, "wide", False),
    (300, 1000, 700, 0.75, "wide", False),
    (300, 1000, 340, 0.97, "fourwave", False),
    (8200, 2000, 200, 0.5, "wide passes=1 nb=1", True),
    (8200, 2000, 256, 0.5, "wide passes=1 nb=1", False),
])
def test_exact(torch, usp, M, K, N, density, route, unaligned):
    W, mask, X = wl.make_small_int(M, K, N, density, seed=M + K + N, lo=-1, hi=1)
    A = usp.SparseMatrix(W, mask)
    plan = A.plan(N)
    print(f"case M={M} K={K} N={N} density={density}: {plan}", flush=True)
    assert plan.startswith(route), plan
    Xd = to_dev(torch, X, 3, 1) if unaligned else to_dev(torch, X)
    ws = A.make_workspace(N)
    rows = np.arange(M)
    if M * K * N > 2 ** 34:  # some rows of every tile
        rows = np.unique(np.concatenate([np.arange(0, M, 61), [M - 1]]))
    Yref, _ = oracle.masked_gemm(W, mask, X, rows=rows)
    for _ in range(2):  # the second call finds the workspace as the first left it
        Y = A.spmm(Xd, workspace=ws)
        torch.cuda.synchronize()
        assert np.array_equal(Y.cpu().numpy().astype(np.float64)[:, rows], Yref)
    assert int(ws[:256 * 1024].count_nonzero().item()) == 0  # arrival counters
    A.free()


# 193 to 256 tokens on a large layer with one nearly dense tile, whose record (7 to
# 8 KB) the wide kernel's ring slots do not hold: the shared-decode kernel.
@pytest.mark.parametrize("M,K,N", [(8200, 2000, 193), (8200, 2000, 256), (28672, 1024, 224)])
def test_one_nearly_dense_tile(torch, usp, M, K, N):
    W, mask, X = wl.make_small_int(M, K, N, 0.5, seed=M + N, lo=-1, hi=1)
    mask[16:32, 256:512] = 1
    mask[16:32, 256:512:10] = 0  # 90% kept
    A = usp.SparseMatrix(W, mask)
    plan = A.plan(N)
    print(f"case M={M} K={K} N={N}: {plan}", flush=True)
    assert plan.startswith("share nb=4") and plan.endswith("pipelined"), plan
    Xd = to_dev(torch, X)
    ws = A.make_workspace(N)
    Y = A.spmm(Xd, workspace=ws)
    bias = torch.ones(M, dtype=torch.float16, device="cuda")
    Yb = A.spmm(Xd, workspace=ws, bias=bias, residual=Y)
    torch.cuda.synchronize()
    A.free()
    Yref, _ = oracle.masked_gemm(W, mask, X)
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), Yref)
    assert np.array_equal(Yb.cpu().numpy().astype(np.float64), (2 * Yref + 1).astype(np.float16))


# 193 to 256 tokens where the device scratch holds the shared-decode plan but not the partials of the wide
# kernel's best plan: the wide kernel on fewer workgroups while they have not much more to do, else the
# shared-decode kernel; usp_spmm_noalloc takes the same route and gives the same bits.
@pytest.mark.parametrize("M,K,N,route", [
    (4096, 11008, 224, "share nb=4 grid=256 pipelined"),
    (8192, 22016, 193, "share nb=4 grid=256 pipelined"),
    (6144, 6144, 200, "wide passes=1 nb=1 grid=192"),
    (5120, 13824, 224, "wide passes=1 nb=1 grid=200"),
    (3584, 8192, 256, "wide passes=1 nb=1 grid=196"),
])
def test_plans_that_the_scratch_limits(torch, usp, M, K, N, route):
    W, mask, X = wl.make_small_int(M, K, N, 0.5, seed=M + N, lo=-1, hi=1)
    A = usp.SparseMatrix(W, mask)
    print(f"case M={M} K={K} N={N}: {A.plan(N)}", flush=True)
    assert A.plan(N) == route and A.workspace_size(N) <= usp.NOALLOC_SCRATCH_BYTES
    Xd = to_dev(torch, X)
    Y = A.spmm(Xd)
    Yn = torch.full_like(Y, float("nan"))
    usp.usp_spmm_noalloc(A.handle, Xd, Yn)
    torch.cuda.synchronize()
    A.free()
    rows = np.unique(np.concatenate([np.arange(0, M, 97), [M - 1]]))
    Yref, _ = oracle.masked_gemm(W, mask, X, rows=rows)
    assert np.array_equal(Y.cpu().numpy().astype(np.float64)[:, rows], Yref)
    assert torch.equal(Yn.view(torch.int16), Y.view(torch.int16))


# The fused epilogue at odd M (no vector stores), residual read from Y itself,
# on a split plan, within the oracle's tolerance.
def test_epilogue_in_place(torch, usp):
    M, K, N = 1101, 900, 330
    W, mask, X = wl.make_random(M, K, N, 0.5, seed=5)
    rng = np.random.default_rng(6)
    bias = rng.normal(0, 0.5, M).astype(np.float16).view(np.uint16)
    res = rng.normal(0, 1.0, (N, M)).astype(np.float16).view(np.uint16)
    A = usp.SparseMatrix(W, mask)
    Y = to_dev(torch, res)
    A.spmm(to_dev(torch, X), Y=Y, bias=to_dev(torch, bias), residual=Y, activation="silu")
    torch.cuda.synchronize()
    A.free()
    Yref, Aref = oracle.masked_gemm(W, mask, X)
    y, scale = oracle.linear_epilogue(Yref, Aref, oracle.ACTIVATIONS["silu"], bias=oracle.f16_to_f64(bias),
                                      residual=oracle.f16_to_f64(res))
    out = oracle.check_tolerance(Y.cpu().numpy().astype(np.float64), y, scale)
    assert out["ok"], out


# Captured in a graph and replayed with eager calls of another handle between,
# all on one workspace.
def test_graph_replays(torch, usp):
    W, mask, X = wl.make_small_int(1100, 700, 400, 0.5, seed=9, lo=-1, hi=1)
    A, B = usp.SparseMatrix(W, mask), usp.SparseMatrix(W[:300], mask[:300])
    Xd = to_dev(torch, X)
    ws = A.make_workspace(400)
    Y = A.spmm(Xd, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        A.spmm(Xd, Y=Y, workspace=ws)
    Yref, _ = oracle.masked_gemm(W, mask, X)
    for _ in range(4):
        Y.fill_(float("nan"))
        Yb = B.spmm(Xd[:60], workspace=ws)
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(Y.cpu().numpy().astype(np.float64), Yref)
        assert np.array_equal(Yb.cpu().numpy().astype(np.float64), Yref[:60, :300])
    A.free()
    B.free()


# Above 256 tokens usp_spmm_noalloc, and usp_spmm with a workspace smaller than usp_workspace_size, run a plan
# that exceeds the workspace in parts of it: the same sums in the same order, so the same bits (weights N(0, 1)).
# Parts of some row sets where ranges cross tiles and where tiles are cut evenly; of some token tiles; of a few
# of a tile's wavefronts (K = 36864: half the scratch holds 220 tokens of X); in two passes, the second shorter;
# unsplit, over tokens alone; X unaligned.
@pytest.mark.parametrize("M,K,N,fraction,unaligned", [
    (4096, 4000, 1024, None, False),
    (5120, 5120, 320, None, False),
    (5433, 2691, 536, None, True),
    (5433, 2691, 536, 0.02, False),
    (5120, 5120, 1500, 0.4, True),
    (300, 36864, 512, None, False),
    (40, 36800, 700, 0.2, True),
    (2000, 3000, 2100, 0.12, False),
    (130, 700, 333, 0.0, True),
])
def test_parts_same_bits(torch, usp, M, K, N, fraction, unaligned):
    g = torch.Generator(device="cuda").manual_seed(M + N)
    W = torch.randn(M, K, generator=g, device="cuda", dtype=torch.float16)
    mask = torch.rand(M, K, generator=g, device="cuda") < 0.5
    A = usp.SparseMatrix(W.cpu().numpy().view(np.uint16), mask.cpu().numpy())
    X = torch.randn(N, K, generator=g, device="cuda", dtype=torch.float16)
    if unaligned:
        buf = torch.empty(N * (K + 3) + 1, dtype=torch.float16, device="cuda")
        Xd = buf[1:].view(N, K + 3)[:, :K]
        Xd.copy_(X)
    else:
        Xd = X
    bias = W[:, 0].contiguous()
    need = A.workspace_size(N)
    print(f"case M={M} K={K} N={N}: {A.plan(N)}, workspace {need} bytes", flush=True)
    assert A.plan(N).startswith("wide")
    part = torch.full((N, M), float("nan"), dtype=torch.float16, device="cuda")
    if fraction is None:
        assert need > usp.NOALLOC_SCRATCH_BYTES
        want = A.spmm(Xd)
        for _ in range(2):  # the second finds the scratch as the first left it
            part.fill_(float("nan"))
            usp.usp_spmm_noalloc(A.handle, Xd, part)
    else:
        want = A.spmm(Xd, bias=bias)
        with pytest.raises(usp.UspError) as e:  # too small for any part
            usp.usp_spmm_ex(A.handle, Xd, part, torch.zeros(256 * 1024, dtype=torch.uint8, device="cuda"), bias)
        assert e.value.status == 1
        ws = None
        for size in range(int(need * fraction) // (256 * 1024) * 256 * 1024, need + 1, 256 * 1024):
            ws = torch.zeros(size, dtype=torch.uint8, device="cuda")
            try:  # the smallest workspace, in steps of 256 KB, that is accepted
                usp.usp_spmm_ex(A.handle, Xd, part, ws, bias)
                break
            except usp.UspError:
                pass
        assert ws.numel() < need
        assert int(ws[:256 * 1024].count_nonzero().item()) == 0
    torch.cuda.synchronize()
    A.free()
    assert torch.equal(part.view(torch.int16), want.view(torch.int16))
    ref = X.float() @ (W * mask).float().t()
    if fraction is not None:
        ref += bias.float()
    assert float((part.float() - ref).norm() / ref.norm()) < 8e-4  # one rounding to fp16: 2.1e-4 measured


# usp_spmm_noalloc where the wide plan exceeds the device scratch, exact.
def test_noalloc_above_scratch(torch, usp):
    W, mask, X = wl.make_small_int(4096, 4000, 1024, 0.5, seed=10, lo=-1, hi=1)
    A = usp.SparseMatrix(W, mask)
    assert A.plan(1024).startswith("wide") and A.workspace_size(1024) > usp.NOALLOC_SCRATCH_BYTES
    Xd = to_dev(torch, X)
    Y = torch.full((1024, A.M), float("nan"), dtype=torch.float16, device="cuda")
    usp.usp_spmm_noalloc(A.handle, Xd, Y)
    torch.cuda.synchronize()
    A.free()
    Yref, _ = oracle.masked_gemm(W, mask, X)
    assert np.array_equal(Y.cpu().numpy().astype(np.float64), Yref)


# Up to 256 tokens: a product whose plan on the shared-decode kernel fits the device scratch (31.6 MB here) and
# whose packed X for the wide kernel alone does not (33.7 MB) is served by usp_spmm_noalloc, with usp_spmm's bits.
def test_noalloc_near_the_scratch(torch, usp):
    M, K, N = 14336, 65280, 225
    rng = np.random.default_rng(12)
    W, mask = np.zeros((M, K), dtype=np.uint16), np.zeros((M, K), dtype=np.uint8)
    rows = np.array([0, 1, 17, 900, M - 17, M - 1])
    for r in rows:
        W[r] = rng.choice(np.array([-1, 0, 1], dtype=np.float16), K).view(np.uint16)
        mask[r] = rng.random(K) < 0.5
    X = rng.choice(np.array([-1, 0, 1], dtype=np.float16), (N, K))
    A = usp.SparseMatrix(W, mask)
    print(f"case M={M} K={K} N={N}: {A.plan(N)}, workspace {A.workspace_size(N)} bytes", flush=True)
    assert A.workspace_size(N) <= usp.NOALLOC_SCRATCH_BYTES
    Xd = torch.from_numpy(X).cuda()
    Y = torch.full((N, M), float("nan"), dtype=torch.float16, device="cuda")
    usp.usp_spmm_noalloc(A.handle, Xd, Y)
    Ys = A.spmm(Xd)
    torch.cuda.synchronize()
    A.free()
    assert torch.equal(Y.view(torch.int16), Ys.view(torch.int16))
    got = Y.cpu().numpy().astype(np.float64)
    Yref, _ = oracle.masked_gemm(W, mask, X.view(np.uint16), rows=rows)
    assert np.array_equal(got[:, rows], Yref)
    assert not np.delete(got, rows, axis=1).any()
