"""The GEMM kernels wait for their memory requests with hand-counted `s_waitcnt vmcnt(N)`.  The build
also makes a library in which every such wait is a wait for everything; both must agree bit for bit,
whatever the compiler did with the instruction order."""
import ctypes

import numpy as np
import pytest

from helpers import STREAMED, TILED, TILED_LINEARS, assert_rows_per_tile, gemm_route
from paper_2504_02658_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _gemm(L, X, q3, U, V, r, N):
    import torch
    M, K = X.shape
    need = int(L.milo_w3lr_gemm_workspace(M, N, K, r))
    ws = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    assert L.milo_workspace_init(ctypes.c_void_p(ws.data_ptr()), ws.numel(), None) == 0
    Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr()) if t is not None else ctypes.c_void_p(0)
    st = L.milo_w3lr_gemm(p(X), M, N, K, p(q3), p(U), p(V), r, p(Y), p(ws), ws.numel(), None)
    assert st == 0
    torch.cuda.synchronize()
    return Y.cpu().numpy()


@pytest.mark.parametrize("M,N,K,r", [
    (16, 1024, 4096, 32), (1, 528, 2112, 16), (4, 272, 14336, 32), (7, 20480, 256, 16), (16, 272, 1408, 20),
    (48, 512, 4096, 24), (130, 528, 1024, 64), (512, 1024, 2048, 8), (16, 1040, 8256, 32), (2, 4096, 14336, 24),
])
def test_counted_waits_equal_full_waits(M, N, K, r):
    import torch
    from paper_2504_02658_amd import api
    counted, full = api.lib(), api.bind(api.FULLWAITS_LIB_PATH)
    rng = np.random.default_rng(M + N + K + r)
    W = torch.from_numpy(wl.gen_weight(N, K, seed=M + N + K)).cuda()
    q3 = api.pack_w3(W).q3
    X = torch.from_numpy(wl.gen_activations(M, K, seed=r + 1)).cuda()
    U = torch.from_numpy((0.02 * rng.standard_normal((N, r))).astype(np.float16)).cuda()
    V = torch.from_numpy((0.02 * rng.standard_normal((r, K))).astype(np.float16)).cuda()
    a = _gemm(counted, X, q3, U, V, r, N)
    b = _gemm(full, X, q3, U, V, r, N)
    assert np.array_equal(a.view(np.uint16), b.view(np.uint16))
    assert np.all(np.isfinite(a)) and np.any(a != 0)


@pytest.mark.parametrize("M,N,K,r,rows,splits", TILED_LINEARS)
@pytest.mark.parametrize("dtype", ["fp16", "symmetric", "bf16", "int3"])
def test_tiled_linear_counted_waits_equal_full_waits(monkeypatch, M, N, K, r, rows, splits, dtype):
    # (above sixteen rows the cases further up take a kernel that counts no waits)
    import torch
    from paper_2504_02658_amd import api
    if dtype == "int3":
        N, r = (N + 63) // 64 * 64, min(r, 128)
        if r == 0 or gemm_route(M, N, K, r, 2)[0] != TILED:
            pytest.skip("no compensator, or not the tiled kernel without ranks above 128")
    else:
        assert gemm_route(M, N, K, r, {"fp16": 0, "symmetric": 1, "bf16": 4}[dtype]) == (TILED, rows, splits)
    g = torch.Generator(device="cuda")
    g.manual_seed(M + N + K + r)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    dt = torch.bfloat16 if dtype == "bf16" else torch.float16
    pw, X = api.pack_w3(randn(N, K) * 0.02, symmetric=dtype == "symmetric"), randn(M, K).to(dt)
    if r:
        U, V = randn(N, r) * 0.1, randn(r, K) * 0.1
        pw = pw.with_int3_compensator(*api.pack_lr3(U, V), r) if dtype == "int3" else pw.with_compensator(U.to(dt), V.to(dt))
    call = lambda: api.w3lr_gemm(X, pw, workspace=api.new_workspace(api.gemm_workspace_bytes(M, N, K, r)))
    Y1 = call()
    with monkeypatch.context() as m:
        m.setattr(api, "_lib", api.bind(api.FULLWAITS_LIB_PATH))
        Y2 = call()
    assert torch.equal(Y1, Y2) and bool(torch.isfinite(Y1.float()).all()) and bool((Y1 != 0).any())


@pytest.mark.parametrize("T,H,F,E,topk,ranks,zipf,rows", [
    # the weight-streaming kernel, three and more chunks per wave in both projections: items of 16 and 4 rows, of 16 and 7,
    # of 3 (the down projection at two row blocks per wave), and a layer whose loop never repeats
    (20, 2304, 2112, 2, 2, (8, 40), 0.0, STREAMED), (23, 2304, 4416, 2, 2, (0, 128), 0.0, STREAMED),
    (3, 4160, 4352, 4, 2, (24,), 0.0, None), (24, 256, 384, 4, 2, (0, 8, 40), 0.0, None),
    # the tiled one at each of its heights, with and without K splits of the down projection
    (80, 1024, 1152, 8, 2, (0, 40, 136), 2.5, 32), (140, 512, 2176, 24, 4, (0, 8, 40), 1.2, 32),
    (160, 1024, 2304, 16, 4, (0, 8, 40), 1.2, 64), (400, 256, 384, 4, 2, (0, 8, 40), 0.0, 128),
])
@pytest.mark.parametrize("dtype", ["fp16", "bf16", "int3"])
def test_moe_layer_counted_waits_equal_full_waits(monkeypatch, T, H, F, E, topk, ranks, zipf, rows, dtype):
    # the grouped kernels of the MoE call count their waits too: the same layer through both builds must agree bit for bit
    import torch
    from paper_2504_02658_amd import api
    less = 0
    if dtype == "int3" and max(ranks) > 128:        # (136 keeps the other types off the streaming kernel, here less room does)
        less, ranks = 256, tuple(min(r, 128) for r in ranks)
    case = wl.MoECase("waits", T=T, H=H, F=F, E=E, topk=topk, seed=41, rank_choices=ranks, zipf_s=zipf)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float16
    g = torch.Generator(device="cuda")
    g.manual_seed(H + F + T)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda")

    def weight(N, K, r):
        pw = api.pack_w3(randn(N, K) * 0.02)
        U, V = randn(N, r) * 0.1, randn(r, K) * 0.1
        if r == 0:
            return pw
        return pw.with_int3_compensator(*api.pack_lr3(U, V), r) if dtype == "int3" else pw.with_compensator(U.to(dt), V.to(dt))

    experts = [tuple(weight(n, k, ranks[e % len(ranks)]) for n, k in ((F, H), (F, H), (H, F))) for e in range(E)]
    X = torch.from_numpy(wl.moe_activations(case)).cuda().to(dt)
    ids_np, gates_np = wl.moe_routing(case)
    ids, gates = torch.from_numpy(ids_np).cuda(), torch.from_numpy(gates_np).cuda()

    def forward():
        layer = api.MoELayer(experts, H, F, bf16=dtype == "bf16")
        ws = api.new_workspace(layer.workspace_bytes(T, topk) - less)
        Y = layer.forward(X, ids, gates, workspace=ws).clone()
        assert layer.routing_status() == 0
        if rows:
            assert_rows_per_tile(layer, ids_np, rows)
        return Y

    Y1 = forward()
    with monkeypatch.context() as m:
        m.setattr(api, "_lib", api.bind(api.FULLWAITS_LIB_PATH))
        Y2 = forward()
    assert torch.equal(Y1, Y2)
    assert bool(torch.isfinite(Y1.float()).all()) and bool((Y1 != 0).any())
