"""GPU parity of milo_w3lr_gemm against the fp64 oracle, all three kernels."""
import numpy as np
import pytest

import oracle
from paper_2504_02658_amd import workloads as wl
from helpers import MID, TILED, TILED_LINEARS, assert_close, gemm_route, oracle_weight, gpu_weight

pytestmark = pytest.mark.gpu


def _run(X, pw):
    import torch
    from paper_2504_02658_amd import api
    return api.w3lr_gemm(torch.from_numpy(X).cuda(), pw).cpu().numpy()


def _check_case(M, N, K, r, seed, outlier_frac=0.0):
    case = wl.LinearCase("t", M=M, N=N, K=K, r=r, seed=seed, outlier_frac=outlier_frac)
    X, W = wl.linear_inputs(case)
    ow = oracle_weight(W, r, seed=seed)
    pw = gpu_weight(W, ow)
    ref = oracle.w3lr_linear(X, **ow)
    Y = _run(X, pw)
    return assert_close(Y, ref, f"M{M} N{N} K{K} r{r}")


def test_c0_small_config():
    c = wl.C0
    _check_case(c.M, c.N, c.K, c.r, c.seed)


@pytest.mark.parametrize("M", [1, 2, 3, 4, 7, 15, 16])
def test_decode_rows(M):
    _check_case(M, 272, 1408, 8, seed=40 + M)          # ragged N (not a multiple of 32), K = 22 groups


@pytest.mark.parametrize("N,K,r", [(16, 64, 0), (48, 192, 8), (1024, 4096, 32), (272, 2112, 24),
                                   (64, 1024, 40), (528, 3136, 16)])
def test_decode_shapes(N, K, r):
    _check_case(16, N, K, r, seed=N + K + r)
    _check_case(5, N, K, r, seed=N + K + r + 1)


@pytest.mark.parametrize("N,K,r", [
    (256, 14336, 32),      # K > 4096: several pieces of 16 chunks per workgroup; staged low-rank path
    (256, 14336, 64),      # the same with more fragments of T
    (20480, 256, 16),      # more row blocks than resident workgroups: second turn of the block loop
    (272, 1408, 20),       # rank not a multiple of 8 at decode: element-wise U loads
    (4096, 14336, 32),     # Mixtral's own down projection at decode (Section 4 shapes)
])
@pytest.mark.parametrize("M", [1, 16])
def test_decode_long_k_many_blocks_odd_rank(N, K, r, M):
    _check_case(M, N, K, r, seed=N + K + r + M)


def test_decode_block_loop_second_turn_with_staged_low_rank():
    # many row blocks with a rank the staged path takes (U fragments are re-copied per turn), and
    # a long K on top of it
    _check_case(16, 36864, 512, 32, seed=811)
    _check_case(3, 16400, 4352, 24, seed=812)


@pytest.mark.parametrize("N,K,r", [
    (64, 8192, 32), (64, 8256, 32),         # four and five fragments of T: one and two chunks per wave of a T worker
    (128, 8192, 128), (80, 10304, 96), (64, 14336, 96), (64, 16384, 128),    # the most fragments that fit the LDS, 16 over 15 waves
    (64, 16448, 128),                       # too many even so: plain rows of T
    (48, 4160, 72),                         # an odd number of rank blocks, the last chunk nearly empty
])
@pytest.mark.parametrize("M", [1, 16])
@pytest.mark.parametrize("dtype", ["fp16", "bf16", "int3"])
def test_decode_parts_of_t(N, K, r, M, dtype):
    import torch
    from paper_2504_02658_amd import api
    if r > N:
        N = (r + 63) // 64 * 64
    if dtype == "int3":
        N = (N + 63) // 64 * 64
    g = torch.Generator()
    g.manual_seed(N + K + r + M)
    randn = lambda *shape: torch.randn(shape, generator=g)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float16
    X, W = randn(M, K).to(dt), (randn(N, K) * 0.02).numpy()
    U, V = randn(N, r) * 0.1, randn(r, K) * 0.1         # a low-rank term larger than the product: its errors show
    q, s, z = oracle.quantize_rtn(W)
    pw = api.pack_w3(torch.from_numpy(W).cuda())
    if dtype == "int3":
        pw = pw.with_int3_compensator(*api.pack_lr3(U.cuda(), V.cuda()), r)
        Ud, Vd = oracle.dequantize_compensator(*oracle.quantize_compensator(U.numpy(), V.numpy()), r)
        if (r + 31) // 32 * ((K + 2047) // 2048) > 16:      # the limit of INT3 compensators at decode sizes
            with pytest.raises(api.MiloError) as e:
                api.w3lr_gemm(X.cuda(), pw)
            assert e.value.status == 2
            return
    else:
        pw = pw.with_compensator(U.to(dt).cuda(), V.to(dt).cuda())
        Ud, Vd = U.to(dt).double().numpy(), V.to(dt).double().numpy()
    Y = api.w3lr_gemm(X.cuda(), pw).double().cpu().numpy()
    ref = oracle.w3lr_linear(X.double().numpy(), q, s, z, Ud, Vd)
    # One rounding to 16 bits in T per K part (their squares add up to one rounding of T), one in the output; fp16 2^-11 each at
    # most, bf16 2^-8, a third of that in the mean.
    assert np.linalg.norm(Y - ref) <= (8.0 if dtype == "bf16" else 1.0) * 2.0 ** -11 * np.linalg.norm(ref)


def _spreads(M, N, K, r, dt):
    """Whether a decode goes to the kernel that hands partial sums over: it writes them behind the workspace's state."""
    import torch
    from paper_2504_02658_amd import api
    zeros = lambda *shape: torch.zeros(shape, dtype=dt, device="cuda")
    pw = api.PackedWeight(N, K, torch.zeros(N * K * 7 // 16, dtype=torch.uint8, device="cuda"))
    if r:
        pw = pw.with_compensator(zeros(N, r), zeros(r, K))
    state = 59648                                               # MILO_WORKSPACE_STATE_BYTES
    ws = api.new_workspace(state + (4 << 20))
    ws[state:] = 0x55
    api.w3lr_gemm(zeros(M, K), pw, workspace=ws)
    assert api.workspace_status(ws) == 0
    return bool((ws[state:] != 0x55).any())


@pytest.mark.parametrize("M,N,K,r,spread", [
    (16, 512, 4352, 0, True),           # 17 chunks: the fewest that are spread over workgroups; 34 of those
    (9, 528, 4160, 20, True),           # the last chunk has 64 columns, the last workgroup's waves past the last pair have none
    (5, 1040, 8256, 128, True),         # eight fragments of T, each band ends in the middle of a workgroup
    (3, 2816, 11008, 24, False),        # chunks in turn (the rule's other side)
    (16, 2816, 11008, 24, True),        # two row blocks per wave
    (2, 12016, 4864, 8, True),          # four, and a band of three at the end
    (1, 1024, 14336, 64, True),         # three partial sums per band
    (7, 528, 65536, 0, True),           # fifteen
    (7, 528, 65536, 16, False),         # T would take all sixteen fragments
    (16, 512, 6144, 32, True),          # every other band starts with a workgroup
    (8, 512, 4160, 0, False), (5, 752, 4160, 48, False),        # a second chunk for few waves only: not worth the hand-over
])
@pytest.mark.parametrize("dtype", ["fp16", "bf16", "int3"])
def test_decode_chunks_spread_over_workgroups(M, N, K, r, spread, dtype):
    import torch
    if r == 0:
        if dtype == "fp16":
            _check_case(M, N, K, r, seed=N + K)
    elif dtype != "int3" or r <= 64:
        test_decode_parts_of_t(N, K, r, M, dtype)
    if dtype != "int3":
        assert _spreads(M, N, K, r, torch.bfloat16 if dtype == "bf16" else torch.float16) == spread


def test_decode_partial_sums_on_a_shared_workspace():
    # partial sums and T carry the launch's number: calls with and without them, other shapes' scratch in between
    _shared_workspace_sequence([
        (16, 1024, 8192, 32), (16, 1024, 8192, 32), (96, 512, 4096, 16), (16, 1024, 8192, 32), (1, 2048, 14336, 0), (4, 256, 1024, 256),
        (1, 2048, 14336, 0), (16, 1024, 8192, 0), (16, 512, 512, 8), (16, 1024, 8192, 32), (300, 256, 1024, 72), (2, 2048, 14336, 0)])


def test_decode_partial_sums_in_scratch_that_looks_like_theirs():
    # every granule holds a value and the mark of the launch that follows; a workspace without room for granules is accepted
    import torch
    from paper_2504_02658_amd import api
    M, N, K, r, state = 16, 1024, 8192, 32, 59648
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    pw = api.pack_w3(randn(N, K) * 0.02).with_compensator((randn(N, r) * 0.1).half(), (randn(r, K) * 0.1).half())
    X = randn(M, K).half()
    ws = api.new_workspace(api.gemm_workspace_bytes(M, N, K, r))
    assert ws.numel() > state
    ref = api.w3lr_gemm(X, pw, workspace=ws)
    for launches in range(1, 5):
        ws[state:].view(torch.int32)[0::2] = 0x42f60000                         # 123.0
        ws[state:].view(torch.int32)[1::2] = launches + 1 - (1 << 31)
        assert torch.equal(api.w3lr_gemm(X, pw, workspace=ws), ref)
    assert api.workspace_status(ws) == 0
    small = api.new_workspace(state)
    Y = api.w3lr_gemm(X, pw, workspace=small)
    assert float((Y.double() - ref.double()).norm() / ref.double().norm()) < 2.0 ** -11       # (another order of the same sums)
    assert api.workspace_status(small) == 0


@pytest.mark.parametrize("M,N,K,r", [(16, 4096, 14336, 32), (16, 512, 512, 0), (512, 1024, 4096, 8), (140000, 64, 64, 8)])
def test_call_without_a_workspace_clears_its_state_and_no_more(M, N, K, r):
    # partial sums and T lie behind the state (here in memory that holds 0x7f.. from before), also the flag words of 140000 rows
    import ctypes
    import torch
    from paper_2504_02658_amd import api
    g = torch.Generator(device="cuda")
    g.manual_seed(13)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    pw = api.pack_w3(randn(N, K) * 0.02)
    if r:
        pw = pw.with_compensator((randn(N, r) * 0.1).half(), (randn(r, K) * 0.1).half())
    X = randn(M, K).half()
    need = max(api.gemm_workspace_bytes(M, N, K, r), 256)
    ref = api.w3lr_gemm(X, pw, workspace=api.new_workspace(need))
    L, cleared = api.lib(), []
    def init(ws, nbytes, stream):
        cleared.append(nbytes)
        return L.milo_workspace_init(ws, nbytes, stream)
    recorder = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p)(init)
    address = lambda f: ctypes.cast(f, ctypes.c_void_p).value
    entries = api._native.entries({n: address(recorder if n == "milo_workspace_init" else getattr(L, n)) for n in api._NATIVE_ENTRIES})
    torch.full((need,), 0x7f, dtype=torch.uint8, device="cuda")                 # (freed at once: the call's own workspace is this memory)
    Y = api._native.gemm(entries, X, pw.q3, pw.U, pw.V, N, K, None, 0, None, None)
    assert torch.equal(Y, ref)
    assert cleared == [min(need, 59648)]                                        # MILO_WORKSPACE_STATE_BYTES


def test_decode_on_a_prefill_workspace_is_the_decode_on_its_own():
    # a workspace for 4096 rows without K splits: 16 rows on it take the kernel that they take with their own, bit for bit
    import torch
    from paper_2504_02658_amd import api
    N, K = 4096, 14336
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    pw = api.pack_w3(torch.randn((N, K), generator=g, device="cuda") * 0.02)
    X = torch.randn((16, K), generator=g, device="cuda").half()
    own, prefill = (api.new_workspace(api.gemm_workspace_bytes(M, N, K, 0)) for M in (16, 4096))
    assert torch.equal(api.w3lr_gemm(X, pw, workspace=own), api.w3lr_gemm(X, pw, workspace=prefill))
    assert api.workspace_status(prefill) == 0


@pytest.mark.parametrize("M", [17, 32, 33, 64, 100, 130, 257])
def test_tiled_rows(M):
    _check_case(M, 272, 1408, 8, seed=60 + M)


@pytest.mark.parametrize("N,K,r", [(16, 64, 0), (48, 192, 8), (528, 1024, 64), (1408, 2048, 128),
                                   (256, 832, 20), (2048, 1408, 136)])
def test_tiled_shapes(N, K, r):
    _check_case(96, N, K, r, seed=N + K + r)


FLAGS = {"fp16": 0, "symmetric": 1, "int3": 2, "bf16": 4}       # of milo.h


def _typed_case(M, N, K, r, dtype):
    """Activations, weight and the oracle's result, with a low-rank term larger than the product: its errors show."""
    import torch
    from paper_2504_02658_amd import api
    g = torch.Generator()
    g.manual_seed(M + N + K + r)
    randn = lambda *shape: torch.randn(shape, generator=g)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float16
    X, W = randn(M, K).to(dt), (randn(N, K) * 0.02).numpy()
    U, V = randn(N, r) * 0.1, randn(r, K) * 0.1
    q, s, z = oracle.quantize_sym(W) if dtype == "symmetric" else oracle.quantize_rtn(W)
    pw = api.pack_w3(torch.from_numpy(W).cuda(), symmetric=dtype == "symmetric")
    Ud, Vd = U.to(dt).double().numpy(), V.to(dt).double().numpy()
    if dtype == "int3":
        pw = pw.with_int3_compensator(*api.pack_lr3(U.cuda(), V.cuda()), r)
        Ud, Vd = oracle.dequantize_compensator(*oracle.quantize_compensator(U.numpy(), V.numpy()), r)
    elif r:
        pw = pw.with_compensator(U.to(dt).cuda(), V.to(dt).cuda())
    return X.cuda(), pw, oracle.w3lr_linear(X.double().numpy(), q, s, z, Ud, Vd)


def _assert_typed_close(Y, ref, dtype):
    # One rounding to 16 bits of each weight, of T and of the output; fp16 2^-11 each at most, bf16 2^-8, a third of that in the mean.
    assert np.linalg.norm(Y.double().cpu().numpy() - ref) <= (8.0 if dtype == "bf16" else 1.0) * 2.0 ** -11 * np.linalg.norm(ref)


@pytest.mark.parametrize("M,N,K,r,form", [
    (17, 16, 64, 8, (32, 1)), (31, 48, 128, 0, (32, 1)), (32, 80, 192, 20, (32, 1)),        # one wave with work, ragged bands and chunks
    (33, 64, 1088, 33, (32, 1)),
    (79, 14336, 1024, 24, (80, 2)), (80, 14400, 1024, 16, (80, 2)), (65, 12816, 1536, 0, (80, 2)),      # the one tile of eighty rows
    (81, 528, 2112, 128, (32, 1)), (160, 1024, 4160, 48, (32, 1)), (257, 272, 1408, 17, (32, 1)),   # several tiles, parts of T that differ in length
    (40, 512, 14336, 64, (32, 1)), (700, 512, 512, 128, (32, 1)),                           # eight parts of T; more than 64 of its blocks
    (64, 14352, 512, 1, (64, 2)), (130, 8208, 704, 40, (32, 2)), (1200, 592, 640, 8, (64, 2)),      # two streams per wave; the most rows
])
@pytest.mark.parametrize("dtype", ["fp16", "symmetric", "bf16", "int3"])
def test_batches_between_decode_and_full_tiles(M, N, K, r, form, dtype):
    import torch
    from paper_2504_02658_amd import api
    if dtype == "int3":
        if r == 0:
            pytest.skip("no compensator")
        N = (N + 63) // 64 * 64
        if (M, N) in ((40, 512), (64, 14400), (130, 8256)):
            pytest.skip("goes to the tiled kernel")
    kind, rows, streams = gemm_route(M, N, K, r, FLAGS[dtype])
    assert kind == MID and ((rows, streams) == form or dtype == "int3")
    X, pw, ref = _typed_case(M, N, K, r, dtype)
    ws = api.new_workspace(api.gemm_workspace_bytes(M, N, K, r))
    Y = api.w3lr_gemm(X, pw, workspace=ws)
    assert torch.equal(api.w3lr_gemm(X, pw, workspace=ws), Y) and api.workspace_status(ws) == 0
    _assert_typed_close(Y, ref, dtype)


@pytest.mark.parametrize("M,N,K,r,rows,splits", TILED_LINEARS)
@pytest.mark.parametrize("dtype", ["fp16", "symmetric", "bf16", "int3"])
def test_tiled_linear(M, N, K, r, rows, splits, dtype):
    # each tile height, with and without K splits, on both sides of the rank limits of the paths that form T (32, 64), odd numbers
    # of groups, ragged rows; what lies behind the state may hold anything; captured calls replay with eager work in between
    import torch
    from paper_2504_02658_amd import api
    if dtype == "int3" and not 0 < r <= 128:
        pytest.skip("no such compensator")
    if dtype == "int3":
        N = (N + 63) // 64 * 64
    assert gemm_route(M, N, K, r, FLAGS[dtype]) == (TILED, rows, splits)
    X, pw, ref = _typed_case(M, N, K, r, dtype)
    ws = api.new_workspace(api.gemm_workspace_bytes(M, N, K, r))
    Y = api.w3lr_gemm(X, pw, workspace=ws).clone()
    _assert_typed_close(Y, ref, dtype)
    ws[59648:].fill_(0xa5)                                      # MILO_WORKSPACE_STATE_BYTES
    out = torch.empty_like(Y)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        api.w3lr_gemm(X, pw, out=out, workspace=ws)
        api.w3lr_gemm(X, pw, out=out, workspace=ws)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, Y)
        assert torch.equal(api.w3lr_gemm(X, pw, workspace=ws), Y)
    assert api.workspace_status(ws) == 0


def test_tiled_linears_on_a_shared_workspace():
    # split sums, T and partials of tiled calls where others keep theirs; M-tiles on both sides of the 128 lines of their words
    _shared_workspace_sequence([
        (31, 64, 12224, 40), (1201, 64, 2112, 40), (77, 256, 1024, 32), (1300, 64, 10048, 64), (16, 1024, 8192, 32), (96, 64, 14272, 20),
        (8192, 64, 512, 40), (8192 + 40, 64, 512, 40), (1201, 128, 12416, 72), (4, 256, 1024, 32), (16384 + 40, 128, 512, 72), (31, 64, 12224, 40)])


@pytest.mark.parametrize("M,N,K,r", [(8, 1024, 1024, 512), (12, 528, 2112, 136), (200, 1024, 1024, 512),
                                     (96, 512, 2048, 300)])
def test_high_rank_compensators(M, N, K, r):
    # ranks of the size the paper gives dense layers (Section 3.2.2, "Dense-512"): beyond what the
    # staged low-rank paths hold at once, so the generic path / several passes over the ranks run
    _check_case(M, N, K, r, seed=500 + M)


@pytest.mark.parametrize("M,N,K,r", [(512, 4096, 4096, 512), (300, 2048, 4096, 1024), (512, 4096, 4096, 200)])
def test_dense_layer_ranks_in_a_split_gemm(M, N, K, r):
    # Dense-512 / Dense-1024 on an attention-sized projection: too few tiles for the chip, so K is split
    # over workgroups; the parts of T share the addition of their partial sums and every K split applies
    # a share of the ranks.  Two runs on one workspace agree bit for bit.
    import torch
    from paper_2504_02658_amd import api
    case = wl.LinearCase("dense", M=M, N=N, K=K, r=r, seed=700 + r)
    X, W = wl.linear_inputs(case)
    ow = oracle_weight(W, r, seed=case.seed)
    pw = gpu_weight(W, ow, check_pack=False)
    ref = oracle.w3lr_linear(X, **ow)
    ws = api.new_workspace(api.gemm_workspace_bytes(M, N, K, r))
    Xd = torch.from_numpy(X).cuda()
    Y1 = api.w3lr_gemm(Xd, pw, workspace=ws).cpu().numpy()
    Y2 = api.w3lr_gemm(Xd, pw, workspace=ws).cpu().numpy()
    assert api.workspace_status(ws) == 0
    assert_close(Y1, ref, f"M{M} N{N} K{K} r{r}")
    assert np.array_equal(Y1.view(np.uint16), Y2.view(np.uint16)), "two runs differ"


def test_rank_zero_equals_no_compensator_and_is_deterministic():
    import torch
    from paper_2504_02658_amd import api
    case = wl.LinearCase("t", M=40, N=512, K=1024, r=16, seed=9)
    X, W = wl.linear_inputs(case)
    ow = oracle_weight(W, 16)
    pw = gpu_weight(W, ow)
    pw0 = api.PackedWeight(pw.N, pw.K, pw.q3)
    for Xm in (X, X[:9]):
        Y0 = _run(Xm, pw0)
        assert_close(Y0, oracle.w3lr_linear(Xm, ow["codes"], ow["scales"], ow["zeros"]), "rank 0")
        Y1a, Y1b = _run(Xm, pw), _run(Xm, pw)
        assert np.array_equal(Y1a.view(np.uint16), Y1b.view(np.uint16)), "two runs differ"
        assert not np.array_equal(Y0, Y1a)


@pytest.mark.parametrize("M", [8, 48])
def test_integer_case_is_exact(M):
    import torch
    from paper_2504_02658_amd import api
    rng = np.random.default_rng(3)
    N, K = 64, 256
    q = rng.integers(0, 8, size=(N, K), dtype=np.uint8)
    s = np.ones((N, K // 64), np.float16)
    z = np.zeros((N, K // 64), np.float16)
    X = rng.integers(-1, 2, size=(M, K)).astype(np.float16)
    pw = api.PackedWeight(N, K, torch.from_numpy(oracle.pack_w3(q, s, z)).cuda())
    Y = _run(X, pw).astype(np.float64)
    assert np.array_equal(Y, oracle.w3lr_linear(X, q, s, z))


@pytest.mark.parametrize("M", [16, 64])
def test_one_hot_activations_expose_the_layout(M):
    # X = rows of the identity: output row k is column k of W_dq + U V, so any permutation of k
    # inside a unit, any swapped plane or transposed compensator shows up element by element.
    N, K, r = 48, 192, 8
    case = wl.LinearCase("t", M=M, N=N, K=K, r=r, seed=77)
    _, W = wl.linear_inputs(case)
    ow = oracle_weight(W, r)
    pw = gpu_weight(W, ow)
    Wt = oracle.dequantize(ow["codes"], ow["scales"], ow["zeros"]) + \
        ow["U"].astype(np.float64) @ ow["V"].astype(np.float64)
    for k0 in range(0, K, M):
        X = np.zeros((M, K), np.float16)
        X[np.arange(M), k0 + np.arange(M)] = 1.0
        Y = _run(X, pw).astype(np.float64)
        ref = Wt[:, k0:k0 + M].T
        assert np.max(np.abs(Y - ref)) <= 2.0 ** -10 * np.max(np.abs(ref)) + 1e-6, f"k0={k0}"


def test_real_valued_zero_points():
    import torch
    from paper_2504_02658_amd import api
    rng = np.random.default_rng(12)
    N, K, r = 128, 512, 0
    q = rng.integers(0, 8, size=(N, K), dtype=np.uint8)
    s = rng.uniform(0.005, 0.03, size=(N, K // 64)).astype(np.float16)
    z = rng.uniform(1.5, 5.5, size=(N, K // 64)).astype(np.float16)
    pw = api.PackedWeight(N, K, torch.from_numpy(oracle.pack_w3(q, s, z)).cuda())
    for M in (4, 40):
        X = rng.standard_normal((M, K)).astype(np.float16)
        assert_close(_run(X, pw), oracle.w3lr_linear(X, q, s, z), f"real z, M={M}")


def test_gpu_int3_compensator_limit():
    # at decode sizes an INT3 compensator takes ceil(r / 32) * ceil(K / 2048) <= 16 fragments of T: rank 128 up
    # to K = 8192, beyond that the call is refused before anything is launched
    import torch
    from paper_2504_02658_amd import api
    rng = np.random.default_rng(7)
    for K, taken in ((8192, True), (8256, False)):
        X = rng.standard_normal((2, K)).astype(np.float16)
        W = (rng.standard_normal((128, K)) * 0.02).astype(np.float32)
        U, V = (rng.standard_normal(s).astype(np.float32) * 0.02 for s in ((128, 128), (128, K)))
        u3, v3 = api.pack_lr3(torch.from_numpy(U).cuda(), torch.from_numpy(V).cuda())
        pw = api.pack_w3(torch.from_numpy(W).cuda()).with_int3_compensator(u3, v3, 128)
        if taken:
            assert api.w3lr_gemm(torch.from_numpy(X).cuda(), pw).shape == (2, 128)
        else:
            with pytest.raises(api.MiloError) as ei:
                api.w3lr_gemm(torch.from_numpy(X).cuda(), pw)
            assert ei.value.status == 2


def test_gpu_argument_errors():
    import torch
    from paper_2504_02658_amd import api
    X = torch.zeros((4, 128), dtype=torch.float16, device="cuda")
    W = torch.zeros((32, 128), dtype=torch.float32, device="cuda")
    pw = api.pack_w3(W)
    with pytest.raises(api.MiloError) as ei:
        api.pack_w3(W, group_size=128)
    assert ei.value.status == 3
    with pytest.raises(api.MiloError) as ei:
        api.w3lr_gemm(X, pw, workspace=torch.zeros(16, dtype=torch.uint8, device="cuda"))
    assert ei.value.status == 5
    with pytest.raises(ValueError):
        api.w3lr_gemm(torch.zeros((4, 64), dtype=torch.float16, device="cuda"), pw)


def test_an_output_that_does_not_fit_raises_out_of_memory():
    # the exception a caller can catch to retry with less; 2^51 bytes (the shape is refused too, but later)
    import torch
    from paper_2504_02658_amd import api
    X = torch.zeros((1 << 20, 64), dtype=torch.float16, device="cuda")
    pw = api.PackedWeight(1 << 30, 64, torch.zeros(448, dtype=torch.uint8, device="cuda"))
    with pytest.raises(torch.OutOfMemoryError):
        api.w3lr_gemm(X, pw)


# ------------------------------------------------------------------ full-size configurations

@pytest.fixture(scope="module")
def c1_weight():
    c = wl.C1[16]
    W = wl.gen_weight(c.N, c.K, c.seed, c.outlier_frac, c.outlier_gain)
    ow = oracle_weight(W, c.r, seed=c.seed)
    pw = gpu_weight(W, ow)
    return ow, pw


@pytest.mark.parametrize("M", [1, 4, 16])
def test_c1_mixtral_up_projection_decode(c1_weight, M):
    ow, pw = c1_weight
    c = wl.C1[M]
    X = wl.gen_activations(c.M, c.K, c.seed)
    assert_close(_run(X, pw), oracle.w3lr_linear(X, **ow), c.name)


def test_c2_mixtral_down_projection_prefill():
    c = wl.C2
    X, W = wl.linear_inputs(c)
    ow = oracle_weight(W, c.r, seed=c.seed)
    pw = gpu_weight(W, ow)
    assert_close(_run(X, pw), oracle.w3lr_linear(X, **ow), c.name)


def test_k_splits_and_t_parts_many_chunks():
    # few tiles and a long K: the whole of it in each workgroup, X V^T in several parts; odd number of groups as well (K splits
    # of the tiled kernel: test_tiled_linear)
    _check_case(48, 512, 4096, 24, seed=301)
    _check_case(200, 256, 8256, 72, seed=302)           # 129 groups


@pytest.mark.parametrize("M,N,K,r", [(16, 528, 2112, 16), (5, 272, 1408, 0), (200, 512, 2048, 24)])
def test_symmetric_weights(M, N, K, r):
    # weights packed by milo_pack_w3_sym (Eq. symm_int3) go through the same kernels
    case = wl.LinearCase("t", M=M, N=N, K=K, r=r, seed=400 + M)
    X, W = wl.linear_inputs(case)
    ow = oracle_weight(W, r, seed=400 + M, symmetric=True)
    pw = gpu_weight(W, ow, symmetric=True)
    assert_close(_run(X, pw), oracle.w3lr_linear(X, **ow), f"symmetric M{M} N{N} K{K} r{r}")


def test_many_m_tiles_take_the_xcd_placement_path():
    # from 128 M-tiles on the tiled kernel renumbers its workgroups (a contiguous share of the
    # tile rows per XCD); with one column tile K is split as well, ragged last tile included
    _check_case(128 * 129 + 40, 256, 2048, 8, seed=303)
    _check_case(128 * 128, 320, 192, 24, seed=304)


def test_graph_replay_matches_eager_and_needs_no_reset():
    # the kernels leave their control words clean: a captured graph of calls that share one
    # workspace per shape can be replayed with eager work in between, bit for bit
    import torch
    from paper_2504_02658_amd import api
    cases = []
    for M, N, K, r, seed in ((16, 1024, 4096, 32, 71), (7, 272, 1408, 8, 72), (96, 512, 4096, 24, 73)):
        case = wl.LinearCase("t", M=M, N=N, K=K, r=r, seed=seed)
        X, W = wl.linear_inputs(case)
        pw = gpu_weight(W, oracle_weight(W, r, seed=seed), check_pack=False)
        Xd = torch.from_numpy(X).cuda()
        ws = api.new_workspace(api.gemm_workspace_bytes(M, N, K, r), Xd.device)
        out = torch.empty((M, N), dtype=torch.float16, device=Xd.device)
        cases.append((Xd, pw, ws, out))
    eager = [api.w3lr_gemm(Xd, pw, workspace=ws).clone() for Xd, pw, ws, _ in cases]
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        for Xd, pw, ws, out in cases:
            api.w3lr_gemm(Xd, pw, out=out, workspace=ws)
    torch.cuda.current_stream().wait_stream(stream)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for _ in range(2):                     # back-to-back calls on the same workspaces
            for Xd, pw, ws, out in cases:
                api.w3lr_gemm(Xd, pw, out=out, workspace=ws)
    for rep in range(3):
        for _, _, _, out in cases:
            out.zero_()
        g.replay()
        torch.cuda.synchronize()
        for (_, _, _, out), ref in zip(cases, eager):
            assert torch.equal(out, ref), f"replay {rep} differs from the eager result"
        # eager work and a synchronisation between the replays
        again = api.w3lr_gemm(cases[0][0], cases[0][1], workspace=cases[0][2])
        torch.cuda.synchronize()
        assert torch.equal(again, eager[0])


def test_workspace_status_reports_a_wait_that_gave_up():
    # The give-up word is forced from the host (no kernel spins): status turns to MILO_ERR_WAIT and
    # stays there until the workspace is prepared again; a clean run reports MILO_OK.
    import torch
    from paper_2504_02658_amd import api
    for M in (16, 96, 1300):                            # workspaces of the three kernels
        assert gemm_route(M, 512, 1024, 16)[0] == {16: 0, 96: MID, 1300: TILED}[M]
        case = wl.LinearCase("t", M=M, N=512, K=1024, r=16, seed=31)
        X, W = wl.linear_inputs(case)
        ow = oracle_weight(W, 16)
        pw = gpu_weight(W, ow, check_pack=False)
        ws = api.new_workspace(api.gemm_workspace_bytes(M, 512, 1024, 16))
        Xd = torch.from_numpy(X).cuda()
        Y = api.w3lr_gemm(Xd, pw, workspace=ws)
        assert api.workspace_status(ws) == 0
        assert_close(Y.cpu().numpy(), oracle.w3lr_linear(X, **ow), "before")
        ws.view(torch.int32)[3] = 1                     # what a kernel writes when its wait runs out
        assert api.workspace_status(ws) == 8
        api.w3lr_gemm(Xd, pw, workspace=ws)
        assert api.workspace_status(ws) == 8            # sticky for a GEMM workspace
        api.lib().milo_workspace_init(ws.data_ptr(), ws.numel(), None)
        Y = api.w3lr_gemm(Xd, pw, workspace=ws)
        assert api.workspace_status(ws) == 0
        assert_close(Y.cpu().numpy(), oracle.w3lr_linear(X, **ow), "after re-init")


def _shared_workspace_sequence(calls):
    """Runs the calls (M, N, K, r) in order on one workspace large enough for all of them; each result has to be, bit for bit,
    what the call gives on a fresh workspace of its own."""
    import torch
    from paper_2504_02658_amd import api
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    made, jobs = {}, []
    for M, N, K, r in calls:
        if (N, K, r) not in made:
            pw = api.pack_w3(randn(N, K) * 0.02)
            if r:
                pw = pw.with_compensator((randn(N, r) * 0.1).half(), (randn(r, K) * 0.1).half())
            made[N, K, r] = pw
        jobs.append((randn(M, K).half(), made[N, K, r]))
    alone = [api.w3lr_gemm(X, pw, workspace=api.new_workspace(api.gemm_workspace_bytes(X.shape[0], pw.N, pw.K, pw.r)))
             for X, pw in jobs]
    ws = api.new_workspace(max(api.gemm_workspace_bytes(*c) for c in calls))
    for (X, pw), ref, call in zip(jobs, alone, calls):
        Y = api.w3lr_gemm(X, pw, workspace=ws)
        assert torch.equal(Y, ref), f"{call} on a workspace that earlier calls used"
    assert api.workspace_status(ws) == 0


def test_calls_of_both_kernels_on_one_workspace():
    # What a call leaves as scratch must not lie where another keeps words that have to be zero at launch: T of decode
    # calls above rank 128, T, partials and split sums of tiled calls, flags of up to and beyond 1024 M-tiles.
    _shared_workspace_sequence([
        (4, 256, 1024, 256), (77, 256, 1024, 32), (4, 256, 1024, 256), (77, 256, 1024, 200), (4096, 256, 1024, 32),
        (16, 256, 1024, 32), (20, 512, 4096, 8), (4096, 256, 1024, 32), (131072 + 40, 16, 64, 8), (96, 512, 4096, 16),
        (131072 + 40, 16, 64, 8), (3, 256, 1024, 256), (131072, 16, 64, 8), (5, 256, 1024, 0), (300, 256, 1024, 72)])


def test_decode_calls_of_many_forms_on_one_workspace():
    # every launch has to move all counters by the same amount, whatever its rank, its parts of T and the number of its
    # streaming workgroups (one, fewer than the 32 counters, a full chip)
    _shared_workspace_sequence([
        (16, 16, 512, 8), (1, 14336, 512, 20), (4, 16, 14336, 16), (16, 1024, 14336, 128), (2, 16, 512, 0), (7, 14336, 512, 8),
        (16, 16, 512, 16), (3, 272, 2048, 128), (8, 528, 4096, 200), (16, 1024, 14336, 128), (5, 14336, 512, 20), (16, 16, 512, 8)])


def test_bytes_behind_the_state_of_a_workspace_may_hold_anything():
    import torch
    from paper_2504_02658_amd import api
    g = torch.Generator(device="cuda")
    g.manual_seed(6)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    state = 59648                                       # MILO_WORKSPACE_STATE_BYTES
    for M, N, K, r in ((4, 256, 1024, 256), (4, 256, 1024, 32), (96, 512, 4096, 24), (131072 + 40, 16, 64, 8)):
        pw = api.pack_w3(randn(N, K) * 0.02).with_compensator((randn(N, r) * 0.1).half(), (randn(r, K) * 0.1).half())
        X = randn(M, K).half()
        ws = api.new_workspace(api.gemm_workspace_bytes(M, N, K, r))
        ref = api.w3lr_gemm(X, pw, workspace=ws)
        ws[state:].fill_(0xa5)
        assert torch.equal(api.w3lr_gemm(X, pw, workspace=ws), ref), (M, N, K, r)
        assert api.workspace_status(ws) == 0


# ------------------------------------------------------------------ INT3 compensators, weight flags

def _int3_case(M, N, K, r, seed, symmetric=False):
    """Both sides of a linear whose compensator is INT3-quantized (Section 3.2.3, Eq. symm_int3)."""
    import torch
    from paper_2504_02658_amd import api
    case = wl.LinearCase("t", M=M, N=N, K=K, r=r, seed=seed)
    X, W = wl.linear_inputs(case)
    ow = oracle_weight(W, r, seed=seed, symmetric=symmetric)
    U32, V32 = ow["U"].astype(np.float32), ow["V"].astype(np.float32)
    uq, vq = oracle.quantize_compensator(U32, V32)
    Ud, Vd = oracle.dequantize_compensator(uq, vq, r)
    ref = oracle.w3lr_linear(X, ow["codes"], ow["scales"], ow["zeros"], Ud, Vd)
    pw = gpu_weight(W, dict(ow, U=np.zeros((N, 0), np.float16)), symmetric=symmetric)
    u3, v3 = api.pack_lr3(torch.from_numpy(U32).cuda(), torch.from_numpy(V32).cuda())
    assert np.array_equal(u3.cpu().numpy(), oracle.pack_w3(*uq)), "U blob differs from the oracle's"
    assert np.array_equal(v3.cpu().numpy(), oracle.pack_w3(*vq)), "V blob differs from the oracle's"
    return X, pw.with_int3_compensator(u3, v3, r), ref


@pytest.mark.parametrize("M,N,K,r", [
    (16, 1024, 4096, 32), (1, 256, 1408, 8), (5, 320, 2112, 20), (16, 4096, 14336, 64), (7, 20480, 256, 16),
    (16, 128, 128, 128), (3, 192, 512, 100),
    (96, 512, 1024, 32), (40, 256, 832, 8), (200, 1024, 2048, 128), (130, 320, 1408, 20), (512, 1024, 4096, 64),
])
def test_int3_compensator(M, N, K, r):
    X, pw, ref = _int3_case(M, N, K, r, seed=M + N + K + r)
    assert pw.flags == 2 and pw.weight_bytes() == (N * K + ((r + 15) // 16 * 16) * (N + K)) * 7 // 16
    assert_close(_run(X, pw), ref, f"INT3 compensator M{M} N{N} K{K} r{r}")


def test_int3_and_bf16_compensators_in_a_split_gemm():
    # rank 128 as INT3 blobs and rank 200 in bf16 on a projection whose K is split over workgroups: the
    # K splits share the ranks, the parts of T share their sums
    import torch
    from paper_2504_02658_amd import api
    X, pw, ref = _int3_case(512, 4096, 4096, 128, seed=901)
    assert_close(_run(X, pw), ref, "INT3 rank 128, split GEMM")
    case = wl.LinearCase("t", M=512, N=4096, K=4096, r=200, seed=902)
    X, W = wl.linear_inputs(case)
    ow = oracle_weight(W, 200, seed=902)
    Xb, Ub, Vb = _to_bf16(X), _to_bf16(ow["U"]), _to_bf16(ow["V"])
    ref = oracle.w3lr_linear(Xb.float().numpy(), ow["codes"], ow["scales"], ow["zeros"], Ub.float().numpy(), Vb.float().numpy())
    pw = gpu_weight(W, dict(ow, U=np.zeros((4096, 0), np.float16)), check_pack=False).with_compensator(Ub.cuda(), Vb.cuda())
    Yf = api.w3lr_gemm(Xb.cuda(), pw).float().cpu().numpy().astype(np.float64)
    rel = np.linalg.norm(Yf - ref) / np.linalg.norm(ref)
    mx = np.max(np.abs(Yf - ref)) / np.max(np.abs(ref))
    assert rel <= BF16_REL_FRO_TOL and mx <= BF16_MAX_ABS_TOL, (rel, mx)


def test_int3_compensator_full_size_c1_and_a_symmetric_weight():
    c = wl.C1[16]
    X, pw, ref = _int3_case(c.M, c.N, c.K, c.r, seed=c.seed)
    assert_close(_run(X, pw), ref, "c1 with INT3 compensator")
    X, pw, ref = _int3_case(16, 1024, 4096, 32, seed=5, symmetric=True)
    assert pw.flags == 3
    assert_close(_run(X, pw), ref, "symmetric weight + INT3 compensator")


@pytest.mark.parametrize("M,N,K,r", [(16, 14336, 4096, 32), (4, 4096, 4096, 0), (16, 272, 1408, 8), (200, 512, 2048, 24)])
def test_symmetric_flag_changes_nothing_but_the_kernel(M, N, K, r):
    # MILO_W3_SYMMETRIC selects the conversion without zero-point arithmetic (Section 3.3): same bits
    import torch
    from paper_2504_02658_amd import api
    case = wl.LinearCase("t", M=M, N=N, K=K, r=r, seed=600 + M)
    X, W = wl.linear_inputs(case)
    rng = np.random.default_rng(M + r)
    pw = api.pack_w3(torch.from_numpy(W).cuda(), symmetric=True)
    assert pw.flags == api.W3_SYMMETRIC
    if r:
        pw = pw.with_compensator(torch.from_numpy((0.02 * rng.standard_normal((N, r))).astype(np.float16)).cuda(),
                                 torch.from_numpy((0.02 * rng.standard_normal((r, K))).astype(np.float16)).cuda())
    plain = api.PackedWeight(pw.N, pw.K, pw.q3, pw.U, pw.V, flags=0)
    a, b = _run(X, pw), _run(X, plain)
    assert np.array_equal(a.view(np.uint16), b.view(np.uint16))


# ------------------------------------------------------------------ bf16 activations (MILO_ACT_BF16)

# Tolerance for the bf16 variant, from its arithmetic: every dequantized weight is rounded once to
# bf16 (relative 2^-9 at most, 2^-9 / sqrt(12) rms; the errors of the K products are independent, so
# they appear undiminished in the relative error of a sum), the output once more, T = X V^T once in
# between: about 1e-3 rms in all, bounded here by 4e-3; single elements by 3e-2 of the largest output.
BF16_REL_FRO_TOL, BF16_MAX_ABS_TOL = 4e-3, 3e-2


def _to_bf16(x):
    import torch
    return torch.from_numpy(np.asarray(x, np.float32)).to(torch.bfloat16)


@pytest.mark.parametrize("M,N,K,r", [(16, 1024, 4096, 32), (1, 272, 1408, 0), (5, 528, 14336, 64), (7, 256, 1408, 20),
                                     (96, 512, 1024, 24), (512, 1024, 4096, 64), (40, 4096, 14336, 16), (130, 272, 832, 136)])
def test_bf16_activations(M, N, K, r):
    import torch
    from paper_2504_02658_amd import api
    case = wl.LinearCase("t", M=M, N=N, K=K, r=r, seed=700 + M + r)
    X, W = wl.linear_inputs(case)
    ow = oracle_weight(W, r, seed=case.seed)
    Xb, Ub, Vb = _to_bf16(X), _to_bf16(ow["U"]), _to_bf16(ow["V"])
    ref = oracle.w3lr_linear(Xb.float().numpy(), ow["codes"], ow["scales"], ow["zeros"],
                             Ub.float().numpy(), Vb.float().numpy())
    pw = gpu_weight(W, dict(ow, U=np.zeros((N, 0), np.float16)))
    if r:
        pw = pw.with_compensator(Ub.cuda(), Vb.cuda())
    Y = api.w3lr_gemm(Xb.cuda(), pw)
    assert Y.dtype == torch.bfloat16
    Yf = Y.float().cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(Yf))
    rel = np.linalg.norm(Yf - ref) / np.linalg.norm(ref)
    mx = np.max(np.abs(Yf - ref)) / np.max(np.abs(ref))
    assert rel <= BF16_REL_FRO_TOL and mx <= BF16_MAX_ABS_TOL, (rel, mx)
    Y2 = api.w3lr_gemm(Xb.cuda(), pw)
    assert torch.equal(Y, Y2)


def test_bf16_integer_case_is_exact():
    # small integers are exact in bf16 too: codes 0..7, scale 1, zero 0, activations in {-1, 0, 1}
    import torch
    from paper_2504_02658_amd import api
    rng = np.random.default_rng(4)
    N, K = 64, 256
    q = rng.integers(0, 8, size=(N, K), dtype=np.uint8)
    s = np.ones((N, K // 64), np.float16)
    z = np.zeros((N, K // 64), np.float16)
    pw = api.PackedWeight(N, K, torch.from_numpy(oracle.pack_w3(q, s, z)).cuda())
    for M in (8, 48):
        X = rng.integers(-1, 2, size=(M, K)).astype(np.float32)
        Y = api.w3lr_gemm(_to_bf16(X).cuda(), pw).float().cpu().numpy().astype(np.float64)
        ref = oracle.w3lr_linear(X, q, s, z)
        assert np.array_equal(Y, np.asarray(_to_bf16(ref).float().numpy(), np.float64))


@pytest.mark.parametrize("M", [16, 64, 128])
def test_bf16_weights_are_rounded_once(M):
    # One-hot rows read the converted weights out: every code at every position of a unit, integer and real-valued
    # zero-points (as the compressor makes them), normal, tiny and large scales.  e s and z s are exact in binary32 (3 and
    # 11 bits times 11), so the weight is the difference rounded to binary32 and then to bf16, bit for bit.
    import torch
    from paper_2504_02658_amd import api
    N, K = 96, 192
    rng = np.random.default_rng(83)
    q = rng.integers(0, 8, size=(N, K)).astype(np.uint8)
    s = (2.0 ** rng.uniform(-14, 6, size=(N, K // 64))).astype(np.float16)
    z = np.where(rng.random((N, K // 64)) < 0.5, rng.integers(0, 8, size=(N, K // 64)), rng.uniform(-12, 20, size=(N, K // 64)))
    z = z.astype(np.float16)
    pw = api.PackedWeight(N, K, torch.from_numpy(oracle.pack_w3(q, s, z)).cuda())
    grow = lambda a: np.repeat(a.astype(np.float64), 64, axis=1)
    want = _to_bf16((q * grow(s) - grow(z) * grow(s)).astype(np.float32))
    for k0 in range(0, K, M):
        rows = torch.zeros(M, K)
        cols = torch.arange(k0, min(k0 + M, K))
        rows[torch.arange(len(cols)), cols] = 1.0
        Y = api.w3lr_gemm(rows.to(torch.bfloat16).cuda(), pw).cpu()
        assert torch.equal(Y[:len(cols)], want[:, cols].T), (M, k0)
