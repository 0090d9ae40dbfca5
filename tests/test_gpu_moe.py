"""GPU parity of milo_moe_w3lr_forward against the fp64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2504_02658_amd import workloads as wl
from helpers import STREAMED, assert_close, assert_rows_per_tile, build_moe

pytestmark = pytest.mark.gpu


def _forward(layer, X, ids, gates, workspace=None):
    import torch
    Y = layer.forward(torch.from_numpy(X).cuda(), torch.from_numpy(ids).cuda(),
                      torch.from_numpy(gates).cuda(), workspace=workspace)
    return Y.cpu().numpy()


def _check(case, what=None, int3=False, rows=None, less=0):
    """rows: the tile height that the batch has to take.  less: bytes that its workspace is short of the size asked for."""
    from paper_2504_02658_amd import api
    o_experts, layer = build_moe(case, int3=int3)
    X = wl.moe_activations(case)
    ids, gates = wl.moe_routing(case)
    ref = oracle.moe_forward(X, o_experts, ids, gates)
    ws = api.new_workspace(layer.workspace_bytes(case.T, ids.shape[1]) - less) if less else None
    Y = _forward(layer, X, ids, gates, ws)
    res = assert_close(Y, ref, what or case.name)
    assert layer.routing_status() == 0
    if rows:
        assert_rows_per_tile(layer, ids, rows)
    Y2 = _forward(layer, X, ids, gates, ws)
    assert np.array_equal(Y.view(np.uint16), Y2.view(np.uint16)), "two runs differ"
    return res


def test_tiny_layer_all_tile_heights():
    base = wl.MoECase("tiny", T=40, H=256, F=384, E=4, topk=2, seed=11, rank_choices=(0, 8, 16))
    _check(base, rows=STREAMED)                               # ~20 rows per expert
    _check(wl.scaled(base, T=80, name="tiny40"))             # ~40 rows
    _check(wl.scaled(base, T=150, name="tiny75"))            # ~75 rows, also streamed: a small layer's weights cost little
    _check(wl.scaled(base, T=400, name="tiny128"), rows=128)  # ~200 rows: 128-row tiles, several per expert


# The tiled kernel at 32- and 64-row tiles: layers that the weight-streaming kernel does not take (a rank above 128, more than
# 512 pairs, or a workspace without room for it), with experts of no, one and several tiles.
TILED = [
    # T, H, F, E, topk, ranks, popularity skew, rows of a tile, bytes the workspace is short of
    (80, 256, 384, 8, 2, (0, 40, 136), 2.5, 32, 0),         # routed by one launch; ranks on both sides of 32 and beyond 128
    (40, 256, 3072, 4, 2, (136,), 2.5, 32, 0),              # K splits of the down projection
    (140, 128, 2176, 24, 4, (0, 8, 40), 1.2, 32, 0),        # the same beyond 512 pairs: the general routing kernels
    (160, 256, 384, 16, 4, (0, 8, 40), 1.2, 64, 0),
    (160, 128, 2176, 16, 4, (0, 8, 40), 1.2, 64, 0),        # with K splits
    (80, 256, 384, 8, 2, (0, 40, 128), 2.5, 32, 256),       # would stream, but for its workspace
]


@pytest.mark.parametrize("T,H,F,E,topk,ranks,zipf,rows,less,dtype", [
    (*c, dtype) for c in TILED for dtype in ("fp16", "bf16", "int3") if dtype != "int3" or max(c[5]) <= 128])
def test_tiled_layer_at_32_and_64_rows(T, H, F, E, topk, ranks, zipf, rows, less, dtype):
    case = wl.MoECase("tiled", T=T, H=H, F=F, E=E, topk=topk, seed=51 + T, rank_choices=ranks, zipf_s=zipf)
    if dtype == "bf16":
        _check_bf16(case, rows=rows, less=less)
    else:
        _check(case, int3=dtype == "int3", rows=rows, less=less)


def test_int3_compensators_in_a_layer():
    # every expert's U, V as INT3 blobs (Section 3.2.3): the grouped kernels unpack them like weights
    base = wl.MoECase("int3", T=40, H=256, F=384, E=4, topk=2, seed=21, rank_choices=(0, 8, 16, 40))
    _check(base, int3=True, rows=STREAMED)
    _check(wl.scaled(base, T=400, name="int3_128", rank_choices=(16, 32, 128)), int3=True, rows=128)


# bfloat16 layer (MILO_ACT_BF16): on top of the single linear's roundings (every dequantized weight, T, the
# output: see test_gpu_gemm) the SwiGLU output and every routed pair's expert output are rounded to bf16
# (2^-9 relative at most, 5.6e-4 rms each) and the second linear sees the first one's error: about 1.3e-3
# rms in all, bounded here by 6e-3; single elements by 4e-2 of the largest output.
BF16_MOE_REL_FRO_TOL, BF16_MOE_MAX_ABS_TOL = 6e-3, 4e-2


def _check_bf16(case, rows=None, less=0):
    import torch
    from helpers import to_bf16
    from paper_2504_02658_amd import api
    o_experts, layer = build_moe(case, bf16=True)
    Xb = to_bf16(wl.moe_activations(case))
    ids, gates = wl.moe_routing(case)
    ref = oracle.moe_forward(Xb.float().numpy(), o_experts, ids, gates)
    args = (Xb.cuda(), torch.from_numpy(ids).cuda(), torch.from_numpy(gates).cuda())
    ws = api.new_workspace(layer.workspace_bytes(case.T, ids.shape[1]) - less) if less else None
    Y = layer.forward(*args, workspace=ws)
    assert Y.dtype == torch.bfloat16
    Yf = Y.float().cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(Yf))
    rel = np.linalg.norm(Yf - ref) / np.linalg.norm(ref)
    mx = np.max(np.abs(Yf - ref)) / np.max(np.abs(ref))
    assert rel <= BF16_MOE_REL_FRO_TOL and mx <= BF16_MOE_MAX_ABS_TOL, (case.name, rel, mx)
    assert layer.routing_status() == 0
    if rows:
        assert_rows_per_tile(layer, ids, rows)
    assert torch.equal(Y, layer.forward(*args, workspace=ws)), "two runs differ"


def test_bf16_layer():
    base = wl.MoECase("bf16", T=40, H=256, F=384, E=4, topk=2, seed=31, rank_choices=(0, 8, 16, 40))
    _check_bf16(base, rows=STREAMED)
    _check_bf16(wl.scaled(base, T=400, name="bf16_128"), rows=128)              # 128-row tiles, several per expert
    _check_bf16(wl.scaled(base, T=3, name="bf16_small"))
    _check_bf16(wl.scaled(wl.C4, T=256, H=512, F=704, E=16, name="bf16_c4_reduced"), rows=128)    # shared experts


def test_bf16_layer_rejects_int3_compensators():
    from paper_2504_02658_amd import api
    case = wl.MoECase("bf16_int3", T=8, H=256, F=384, E=2, topk=1, seed=32, rank_choices=(16,))
    _, layer = build_moe(case, int3=True)
    with pytest.raises(api.MiloError) as ei:
        api.MoELayer(layer.experts, case.H, case.F, bf16=True)
    assert ei.value.status == 2


def test_many_tiles_take_the_xcd_placement_path():
    # 16 800 routed rows -> more than 128 M-tiles: the grouped kernels renumber their workgroups
    # per XCD and the work list is dealt over the eight ranges
    case = wl.MoECase("many", T=4200, H=256, F=384, E=8, topk=4, seed=14, rank_choices=(0, 8, 24))
    _check(case)


def test_rows_wider_than_the_layer_are_refused():
    """The call goes by the activations' own width, for which the layer's workspace is too small."""
    import torch
    from paper_2504_02658_amd import api
    case = wl.MoECase("wide", T=64, H=256, F=384, E=4, topk=2, seed=13, rank_choices=(0, 8))
    _, layer = build_moe(case)
    ids, gates = (torch.from_numpy(a).cuda() for a in wl.moe_routing(case))
    wide = torch.zeros((case.T, 4 * case.H), dtype=torch.float16, device="cuda")
    with pytest.raises(api.MiloError) as e:
        layer.forward(wide, ids, gates)
    assert e.value.status == 5                                # MILO_ERR_WORKSPACE


def test_rows_of_another_width_are_refused_whatever_the_workspace_holds():
    # a workspace that earlier, larger forwards have grown has room for a few rows of any width
    import torch
    from paper_2504_02658_amd import api
    case = wl.MoECase("widths", T=512, H=256, F=384, E=4, topk=2, seed=14, rank_choices=(0, 8))
    _, layer = build_moe(case)
    ids, gates = (torch.from_numpy(a).cuda() for a in wl.moe_routing(case))
    X = torch.randn((case.T, case.H), device="cuda").half()
    ref = layer.forward(X, ids, gates)
    assert layer._ws.numel() > layer.workspace_bytes(4, case.topk) * 8
    for width, status in ((2 * case.H, 5), (case.H + 64, 5), (case.H - 64, 2)):
        rows = torch.zeros((4, width), dtype=torch.float16, device="cuda")
        for ws in (None, layer._ws):
            with pytest.raises(api.MiloError) as e:
                layer.forward(rows, ids[:4], gates[:4], workspace=ws)
            assert e.value.status == status
    with pytest.raises(ValueError):
        layer.forward(X, ids[:-1].contiguous(), gates)
    with pytest.raises(ValueError):
        layer.forward(X, ids, gates[:-1].contiguous())
    # more routing rows than tokens are fine: the first T count
    assert torch.equal(layer.forward(X[:100], ids, gates), layer.forward(X[:100], ids[:100], gates[:100]))
    assert torch.equal(layer.forward(X, ids, gates), ref)


@pytest.mark.parametrize("T,E,topk,ranks,zipf,rows", [
    (150, 4, 2, (8, 16), 0.0, STREAMED),
    (80, 8, 2, (8, 136), 2.5, 32),          # the tiled kernel's flags, single-launch routing
    (160, 16, 4, (8, 16), 1.2, 64),         # and the general one
    (300, 4, 2, (8, 16), 0.0, 128),
])
def test_graph_replay_of_a_layer(T, E, topk, ranks, zipf, rows):
    # routing, flags and partial buffers are re-initialised by the kernels themselves: a captured
    # layer replays bit for bit with eager work on the same workspace in between
    import torch
    case = wl.MoECase("replay", T=T, H=256, F=384, E=E, topk=topk, seed=15, rank_choices=ranks, zipf_s=zipf)
    _, layer = build_moe(case)
    X = torch.from_numpy(wl.moe_activations(case)).cuda()
    ids_np, gates_np = wl.moe_routing(case)
    ids, gates = torch.from_numpy(ids_np).cuda(), torch.from_numpy(gates_np).cuda()
    from paper_2504_02658_amd import api
    ws = api.new_workspace(layer.workspace_bytes(case.T, case.topk), X.device)
    out = torch.empty((case.T, case.H), dtype=torch.float16, device=X.device)
    eager = layer.forward(X, ids, gates, workspace=ws).clone()
    assert_rows_per_tile(layer, ids_np, rows)
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        layer.forward(X, ids, gates, out=out, workspace=ws)
    torch.cuda.current_stream().wait_stream(stream)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        layer.forward(X, ids, gates, out=out, workspace=ws)
        layer.forward(X, ids, gates, out=out, workspace=ws)
    for rep in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager), f"replay {rep} differs from the eager result"
        again = layer.forward(X, ids, gates, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(again, eager)


def test_single_token_and_empty_experts():
    case = wl.MoECase("one", T=1, H=128, F=192, E=8, topk=2, seed=12, rank_choices=(8,))
    _check(case)                                              # six experts receive nothing


def test_shared_experts_and_skew():
    case = wl.scaled(wl.C4, T=200, H=256, F=320, E=16, topk=4, name="ds_small", shared_rank=24)
    _check(case)


def test_reduced_mixtral_and_deepseek_shapes():
    _check(wl.scaled(wl.C3, T=96, H=512, F=1792, name="c3_reduced"))
    _check(wl.scaled(wl.C4, T=512, H=512, F=704, E=24, name="c4_reduced"))


def test_out_of_range_expert_id_is_skipped_and_flagged():
    case = wl.MoECase("bad", T=24, H=128, F=192, E=4, topk=2, seed=13, rank_choices=(8,))
    o_experts, layer = build_moe(case)
    X = wl.moe_activations(case)
    ids, gates = wl.moe_routing(case)
    ids = ids.copy()
    ids[5, 1] = 4
    ids[7, 0] = -1
    good = (ids >= 0) & (ids < 4)
    ref = oracle.moe_forward(X, o_experts, np.where(good, ids, 0), np.where(good, gates, 0).astype(np.float32))
    Y = _forward(layer, X, ids, gates)
    assert_close(Y, ref, "bad ids skipped")
    assert layer.routing_status() == 6


def test_status_reports_a_wait_that_gave_up():
    # the give-up word of the layer's workspace, forced from the host (no kernel spins): the status call
    # reports MILO_ERR_WAIT for that forward; the next forward clears the word at its start
    import torch
    from paper_2504_02658_amd import api
    case = wl.MoECase("wait", T=24, H=128, F=192, E=4, topk=2, seed=16, rank_choices=(8,))
    _, layer = build_moe(case)
    X = torch.from_numpy(wl.moe_activations(case)).cuda()
    ids_np, gates_np = wl.moe_routing(case)
    ids, gates = torch.from_numpy(ids_np).cuda(), torch.from_numpy(gates_np).cuda()
    ws = api.new_workspace(layer.workspace_bytes(case.T, case.topk))
    Y = layer.forward(X, ids, gates, workspace=ws).clone()
    assert layer.routing_status() == 0
    ws.view(torch.int32)[3] = 1                         # what a kernel writes when its wait runs out
    assert layer.routing_status() == 8
    Y2 = layer.forward(X, ids, gates, workspace=ws)
    assert layer.routing_status() == 0
    assert torch.equal(Y, Y2)


@pytest.mark.timeout(900)
def test_c3_mixtral_layer_full_size():
    # the full layer at 512 tokens (128-row tiles), then the same experts at decode-sized batches (64 tokens:
    # 32-row tiles with K splits of the down projection; 16, 4 and 1: the weight-streaming kernel)
    import dataclasses
    import torch
    o_experts, layer = build_moe(wl.C3)
    for T, rows in ((512, 128), (64, 32), (16, None), (4, None), (1, None)):
        case = dataclasses.replace(wl.C3, T=T)
        X = wl.moe_activations(case)
        ids, gates = wl.moe_routing(case)
        ref = oracle.moe_forward(X, o_experts, ids, gates)
        Y = _forward(layer, X, ids, gates)
        assert_close(Y, ref, f"c3 at {T} tokens")
        assert layer.routing_status() == 0
        if rows == 128:
            assert_rows_per_tile(layer, ids, rows)
        elif rows:                  # (no expert has more than 32 rows here: any height but the streamed items' fits)
            n = np.bincount(ids.ravel(), minlength=layer.E)
            assert int(layer.last_workspace.view(torch.int32)[1]) == int(np.sum((n + 31) // 32)) != int(np.sum((n + 15) // 16))
        Y2 = _forward(layer, X, ids, gates)
        assert np.array_equal(Y.view(np.uint16), Y2.view(np.uint16)), "two runs differ"


def test_routing_of_small_batches_matches_the_general_kernels():
    # up to 512 routed pairs (and experts) the routing and the work list of 32-row tiles come from one single-workgroup
    # kernel, from 513 on from the two general kernels: the same tokens below and above the limit give the same bits (a
    # row's result does not depend on the tile it lands in), with many experts empty, several tiles per expert, ranks on
    # both sides of 32 and ids out of range; the same layer's few-row batches beside it
    import torch
    base = wl.MoECase("small_route", T=64, H=128, F=192, E=24, topk=4, seed=23, rank_choices=(0, 8, 40))
    _check(base, rows=STREAMED)
    _check(wl.scaled(base, T=3, name="three_tokens"))
    case = wl.MoECase("general_route", T=129, H=256, F=192, E=24, topk=4, seed=53, rank_choices=(0, 8, 40, 136), zipf_s=1.2)
    o_experts, layer = build_moe(case)
    X = wl.moe_activations(case)
    ids, gates = wl.moe_routing(case)
    ids = ids.copy()
    ids[3, 1], ids[77, 0], ids[127, 3] = -1, case.E, 1 << 20
    good = (ids >= 0) & (ids < case.E)
    ref = oracle.moe_forward(X, o_experts, np.where(good, ids, 0), np.where(good, gates, 0).astype(np.float32))
    general = _forward(layer, X, ids, gates)                  # 516 pairs
    assert_close(general, ref, "general routing")
    assert_rows_per_tile(layer, ids, 32)
    assert layer.routing_status() == 6
    small = _forward(layer, X[:128], ids[:128], gates[:128])  # 512
    assert layer.routing_status() == 6
    assert_rows_per_tile(layer, ids[:128], 32)
    assert np.array_equal(general[:128].view(np.uint16), small.view(np.uint16))


@pytest.mark.parametrize("rank", [8, 136])
@pytest.mark.parametrize("E,topk,T", [(5, 2, 16), (5, 2, 17), (5, 1, 33), (3, 3, 21), (3, 3, 22), (200, 4, 127), (200, 4, 128), (511, 1, 512), (512, 8, 64)])
def test_single_launch_routing_at_its_edges(E, topk, T, rank):
    # 32 and 33 pairs (one count per thread, one per wave), 63 to 66 (one wave and a second), 508 and 512, the last expert ids;
    # streamed items and tiles: each row against the row alone, which is routed by itself
    import torch
    from paper_2504_02658_amd import api
    H, F = 192, 192
    g = torch.Generator(device="cuda")
    g.manual_seed(E + T + rank)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    kinds = [tuple(api.pack_w3(randn(n, k) * 0.05).with_compensator((randn(n, r) * 0.1).half(), (randn(r, k) * 0.1).half())
                   for n, k in ((F, H), (F, H), (H, F))) for r in (8, rank, 40)]
    layer = api.MoELayer([kinds[(7 * e) % 3] for e in range(E)], H, F)
    X = randn(T, H).half()
    ids = torch.rand((T, E), generator=g, device="cuda").argsort(dim=1)[:, :topk].to(torch.int32).contiguous()
    ids[0, 0] = E - 1                                       # (may name an expert twice: both rows count)
    ids[T - 1, topk - 1] = 0
    gates = torch.rand((T, topk), generator=g, device="cuda")
    Y = layer.forward(X, ids, gates).clone()
    assert layer.routing_status() == 0
    rows = layer.last_workspace.view(torch.int32)[1].item()
    n = np.bincount(ids.cpu().numpy().ravel(), minlength=E)
    assert rows == int(np.sum((n + (31 if rank > 128 else 15)) // (32 if rank > 128 else 16)))
    for t in range(0, T, 1 if T < 64 else 29):
        alone = layer.forward(X[t:t + 1].clone(), ids[t:t + 1].clone(), gates[t:t + 1].clone())
        assert torch.equal(alone[0], Y[t]), t


def test_single_launch_routing_of_many_tiles():
    # 512 pairs over 220 experts: more than 128 tiles, whose list the tiled kernel reads as eight ranges
    _check(wl.MoECase("many_small", T=128, H=256, F=192, E=220, topk=4, seed=56, rank_choices=(8, 136), zipf_s=0.4), rows=32)


@pytest.mark.parametrize("E,topk,T", [
    (5, 3, 683), (5, 1, 4095), (66, 2, 2049),           # ids that end within a lane's four; one step of 4096 pairs, and two
    (40, 8, 4096), (40, 8, 4097), (3, 1, 40001),        # eight steps, which stay in registers, and more
    (1500, 6, 700),                                     # more slots than a wave of the ordering kernel takes at once
])
def test_routing_by_steps(E, topk, T):
    import torch
    from paper_2504_02658_amd import api
    g = torch.Generator(device="cuda")
    g.manual_seed(E + T)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    kinds = [tuple(api.pack_w3(randn(64, 64) * 0.1) for _ in range(3)) for _ in range(3)]
    layer = api.MoELayer([kinds[e % 3] for e in range(E)], 64, 64)
    X = randn(T, 64).half()
    ids = torch.argsort(torch.rand((T, E), generator=g, device="cuda"), dim=1)[:, :topk].to(torch.int32).contiguous()
    ids[T // 2, 0], ids[T - 1, topk - 1] = -1, E + 5
    gates = torch.rand((T, topk), generator=g, device="cuda")
    Y = layer.forward(X, ids, gates).double()
    assert layer.routing_status() == 6
    # the three experts there are, dequantized by the library (tested by itself), in 64 bits; H and each pair's output are 16-bit
    w = [[api.dequant_w3(p).double() for p in k] for k in kinds]
    x, ref = X.double(), torch.zeros((T, 64), dtype=torch.float64, device="cuda")
    out = [(torch.nn.functional.silu(x @ a.T) * (x @ b.T)) @ c.T for a, b, c in w]
    for j in range(topk):
        good = (ids[:, j] >= 0) & (ids[:, j] < E)
        for k in range(3):
            ref += torch.where((good & (ids[:, j] % 3 == k))[:, None], gates[:, j, None].double() * out[k], 0.0)
    # every row by itself: a pair that went astray is an error of the size of the row; roundings are 2^-11 of it each
    err = (Y - ref).norm(dim=1) / ref.norm(dim=1).clamp_min(1e-6)
    assert float(err[ref.norm(dim=1) > 1e-3].max()) < 6 * 2.0 ** -11
    assert float(Y[ref.norm(dim=1) == 0].abs().sum()) == 0.0


@pytest.mark.timeout(900)
def test_c4_deepseek_layer_full_size():
    _check(wl.C4)


@pytest.mark.parametrize("H,F,E,topk,T,ranks", [
    (64, 64, 2, 1, 1, (0,)),                    # one chunk for four waves, one band
    (192, 128, 4, 2, 7, (8, 20)),               # a chunk that is not whole, elementwise U rows
    (320, 1408, 3, 3, 16, (16, 40)),            # every expert sixteen rows: one full item each; odd numbers of rank blocks
    (320, 320, 3, 3, 17, (8, 24)),              # seventeen: a second item of one row
    (576, 4224, 5, 2, 9, (0, 64, 128)),         # K parts of T in the down projection, more fragments than waves
    (4352, 256, 6, 2, 20, (32,)),               # K parts of T in the gate and up projections
    (128, 192, 512, 1, 512, (8,)),              # largest batch and expert table of the single-launch routing
    (128, 192, 40, 8, 64, (0, 8)),              # 512 pairs, a few items per expert
])
@pytest.mark.parametrize("dtype", ["fp16", "bf16", "int3"])
def test_few_rows_per_expert(H, F, E, topk, T, ranks, dtype):
    # the weight-streaming kernel of decode-sized batches at the edges of its tiles
    case = wl.MoECase("few", T=T, H=H, F=F, E=E, topk=topk, seed=H + F + T, rank_choices=ranks)
    if dtype == "bf16":
        _check_bf16(case)
    else:
        _check(case, int3=dtype == "int3")


@pytest.mark.parametrize("dtype", ["fp16", "bf16"])
def test_a_row_does_not_depend_on_the_height_of_its_tile(dtype):
    # 560 pairs in 32-row tiles, the same tokens among ten times as many in 128-row tiles: T = X V^T is read from memory, or staged
    # with ranks up to 32, and every sum has one order
    import torch
    from paper_2504_02658_amd import api
    E, H, F, dt = 24, 1088, 384, torch.bfloat16 if dtype == "bf16" else torch.float16
    g = torch.Generator(device="cuda")
    g.manual_seed(8)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    experts = [tuple(api.pack_w3(randn(n, k) * 0.05).with_compensator((randn(n, r) * 0.1).to(dt), (randn(r, k) * 0.1).to(dt))
                     for n, k in ((F, H), (F, H), (H, F))) for r in (8, 24, 32, 40) * 6]
    layer = api.MoELayer(experts, H, F, bf16=dtype == "bf16")
    X = randn(1400, H).to(dt)
    ids = torch.rand((1400, E), generator=g, device="cuda").argsort(dim=1)[:, :4].to(torch.int32).contiguous()
    ids[:40, 0] = 0                                         # more than 32 rows of one expert: several tiles
    gates = torch.rand((1400, 4), generator=g, device="cuda")
    tall = layer.forward(X, ids, gates).clone()
    assert_rows_per_tile(layer, ids.cpu().numpy(), 128)
    low = layer.forward(X[:140].clone(), ids[:140].clone(), gates[:140].clone())
    assert_rows_per_tile(layer, ids[:140].cpu().numpy(), 32)
    assert torch.equal(low, tall[:140])


@pytest.mark.parametrize("T", [20, 600])      # streamed, 128-row tiles
def test_swiglu_at_the_ends_of_its_range(T):
    # Gates from -88.5 to 88.5, up projections of 2^100: below a gate of -87.3 the quotient's denominator is above 2^126, its reciprocal
    # below the normal numbers and the product a normal number still.  Every feature of the SwiGLU output is copied to the layer's output.
    import torch
    from paper_2504_02658_amd import api
    H = F = 192
    n, codes = np.arange(F), np.zeros((3, F, H), np.uint8)
    scales = np.zeros((3, F, 3), np.float16)
    codes[0, :, 64], scales[0, :, 1] = 1, np.where(n < 177, 0.5 * (n + 1), 1.0)         # gate: X[64] times 0.5 .. 88.5
    codes[1, :, 0], scales[1, :, 0] = 1, 1.0                                            # up: X[0]
    codes[2, n, n], scales[2] = 1, 1.0
    w = [api.PackedWeight(F, H, torch.from_numpy(oracle.pack_w3(c, s, np.zeros((F, 3), np.float16))).cuda()) for c, s in zip(codes, scales)]
    layer = api.MoELayer([tuple(w)], H, F, bf16=True)
    X = torch.zeros((T, H), dtype=torch.bfloat16, device="cuda")
    X[:, 0] = 2.0 ** 100
    X[:, 64] = torch.tensor([-1.0, 1.0, -0.5, 0.0], device="cuda").repeat((T + 3) // 4)[:T].to(torch.bfloat16)
    ids, gates = torch.zeros((T, 1), dtype=torch.int32, device="cuda"), torch.ones((T, 1), device="cuda")
    Y = layer.forward(X, ids, gates).double().cpu()
    assert_rows_per_tile(layer, ids.cpu().numpy(), STREAMED if T == 20 else 128)
    a = X[:, 64].double().cpu()[:, None] * torch.from_numpy(scales[0, :, 1].astype(np.float64))
    ref = a / (1.0 + torch.exp(-a)) * 2.0 ** 100
    # two roundings to bf16, 2^-9 of the value each; the exponential's argument is rounded to fp32, 88 * 2^-24 of the result
    assert bool(((Y - ref).abs() <= (2.0 ** -8 + 2.0 ** -16) * ref.abs()).all())


def test_few_rows_routing_rejects_and_repeats():
    # ids out of range leave no item behind, and an expert named twice by a token gets both rows
    case = wl.MoECase("few_ids", T=6, H=128, F=192, E=4, topk=3, seed=29, rank_choices=(8,))
    o_experts, layer = build_moe(case)
    X = wl.moe_activations(case)
    _, gates = wl.moe_routing(case)
    ids = np.array([[0, 0, 0], [1, 4, 1], [-1, 2, 2], [7, -3, 9], [2, 2, 2], [0, 1, 2]], np.int32)
    good = (ids >= 0) & (ids < 4)
    ref = oracle.moe_forward(X, o_experts, np.where(good, ids, 0), np.where(good, gates, 0).astype(np.float32))
    assert_close(_forward(layer, X, ids, gates), ref, "repeated and bad ids")
    assert layer.routing_status() == 6


def test_workspace_of_a_larger_batch_serves_smaller_ones():
    # 250 tokens take the weight-streaming kernel and 260 the tiled one, which needs less room: a workspace sized for
    # 260 has room for 250, one of two thirds of that is accepted (by the tiled kernel, 128-row tiles), and one too small for
    # both is not
    import torch
    from paper_2504_02658_amd import api
    case = wl.MoECase("ws", T=250, H=1024, F=512, E=8, topk=2, seed=37, rank_choices=(32,))
    o_experts, layer = build_moe(case)
    X, (ids, gates) = wl.moe_activations(case), wl.moe_routing(case)
    args = [torch.from_numpy(a).cuda() for a in (X, ids, gates)]
    need = layer.workspace_bytes(250, 2)
    assert layer.workspace_bytes(260, 2) >= need
    ws = api.new_workspace(2 * need // 3)
    ref = oracle.moe_forward(X, o_experts, ids, gates)
    for workspace in (ws, None, ws):
        assert_close(layer.forward(*args, workspace=workspace).cpu().numpy(), ref, "workspace of a larger batch")
        assert layer.routing_status() == 0
    # (on any workspace of at least the size asked for the bits are the same)
    assert torch.equal(layer.forward(*args), layer.forward(*args, workspace=api.new_workspace(layer.workspace_bytes(260, 2))))
    with pytest.raises(api.MiloError):
        layer.forward(*args, workspace=api.new_workspace(65536))


def test_few_rows_parts_of_t_are_added_in_fp32():
    # Two K parts of T in the down projection that nearly cancel: the halves of H are equal and V's second half is the first
    # one's negative, up to four columns, so |T| is about |part| / 32.  Rounding the parts to 16 bits would leave
    # an error of about 32 * 2^-12 = 8e-3; rounding H, T and the output, 2^-11 at most each, is 1.5e-3, plus H's own
    # products (16-bit weights, fp32 sums): 2e-3.
    import torch
    from paper_2504_02658_amd import api
    H, F, T, r = 128, 8192, 5, 16
    g = torch.Generator(device="cuda")
    g.manual_seed(41)
    randn = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    w1, w3 = (api.pack_w3(torch.cat([w, w])) for w in (randn(F // 2, H) * 0.1, randn(F // 2, H) * 0.1))
    v = randn(r, F // 2).half()
    v2 = -v
    v2[:, 5::1024] = 0
    U, V = randn(H, r).half(), torch.cat([v, v2], dim=1).contiguous()
    w2 = api.pack_w3(randn(H, F) * 1e-4)
    X = randn(T, H).half()
    ids, gates = torch.zeros(T, 1, dtype=torch.int32, device="cuda"), torch.ones(T, 1, device="cuda")
    Y = api.MoELayer([(w1, w3, w2.with_compensator(U, V))], H, F).forward(X, ids, gates)
    d = lambda pw: api.dequant_w3(pw).double().cpu()
    a, b = X.double().cpu() @ d(w1).T, X.double().cpu() @ d(w3).T
    h = a * torch.sigmoid(a) * b
    low = (h @ V.double().cpu().T) @ U.double().cpu().T
    ref = h @ d(w2).T + low
    assert float(low.norm()) > 10 * float((ref - low).norm())
    assert float((Y.double().cpu() - ref).norm() / ref.norm()) < 2e-3
