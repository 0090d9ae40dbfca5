"""Workloads of the compensated W3A16 linear, the MoE layer, the packer and the compressor, as a program
that uses them calls them.

Each case is one pass through the public calls of paper_2504_02658_amd.api on inputs that are resident on the
GPU: a call (or a chain of calls, one per layer of a model) of w3lr_gemm with the workspace and the outputs a
serving program keeps, one forward of an MoELayer, pack_w3 of a weight, or compress_w3lr of a weight.  Sizes are
those of workloads.py, bench.py and the tests: expert FFN matrices of Mixtral-8x7B (hidden 4096, ffn 14336) and
of a DeepSeek-MoE-style layer (hidden 2048, 64 + 2 experts of ffn 1408), plus generic ones in between.
"""
import math

import torch

from paper_2504_02658_amd import api, workloads as wl

CALIBRATION_ROWS = 256
GROUP_BITS = 3.5            # packed bits per weight: 3 of code, two fp16 parameters per group of 64


def _linear(M, N, K, r, dtype="fp16", symmetric=False, int3=False, layers=1):
    return dict(kind="linear", M=M, N=N, K=K, r=r, dtype=dtype, symmetric=symmetric, int3=int3, layers=layers)


def _moe(T, H, F, E, topk, ranks, shared=0, shared_rank=0, zipf=0.0, dtype="fp16"):
    return dict(kind="moe", T=T, H=H, F=F, E=E, topk=topk, ranks=ranks, shared=shared, shared_rank=shared_rank,
                zipf=zipf, dtype=dtype)


def listed():
    cases = [
        # The smallest call: a 1024 x 1024 projection at a decode batch of 16.  All latency.
        ("decode_small", _linear(16, 1024, 1024, 16)),
        # Decode of 16 sequences through the up projections of eight successive layers: every weight comes
        # from HBM, as it does in a model that is larger than the caches.
        ("decode_up_16", _linear(16, 14336, 4096, 32, layers=8)),
        # Decode of one sequence in bf16 through the down projections (long K) of eight layers.
        ("decode_down_1_bf16", _linear(1, 4096, 14336, 32, dtype="bf16", layers=8)),
        # A small batch of ragged size (speculative or batched decode) on symmetric weights whose
        # compensators are stored as INT3, the smallest form a model takes.
        ("batch_77_sym_int3", _linear(77, 14336, 4096, 32, symmetric=True, int3=True)),
        # Prefill of 512 tokens through a down projection.
        ("prefill_down_512", _linear(512, 4096, 14336, 64)),
        # A long prompt in bf16 through an up projection.
        ("prefill_up_4096_bf16", _linear(4096, 14336, 4096, 32, dtype="bf16")),
        # A Mixtral-shaped layer at a decode batch of 16 tokens, and at a prefill of 512.
        ("moe_mixtral_16", _moe(16, 4096, 14336, 8, 2, "16,32,64")),
        ("moe_mixtral_512", _moe(512, 4096, 14336, 8, 2, "16,32,64")),
        # A DeepSeek-MoE-shaped layer (many small experts, two always-on ones with a high rank, skewed
        # popularity) at a decode batch of 4 tokens in bf16, and at a prefill of 4096.
        ("moe_deepseek_4_bf16", _moe(4, 2048, 1408, 64, 6, "8", shared=2, shared_rank=128, zipf=1.2, dtype="bf16")),
        ("moe_deepseek_4096", _moe(4096, 2048, 1408, 64, 6, "8", shared=2, shared_rank=128, zipf=1.2)),
        # Round-to-nearest quantization and packing of one expert weight.
        ("pack_up", dict(kind="pack", N=14336, K=4096, symmetric=False)),
        # One-shot compression (offline) of the same weight: half-quadratic zero-points, then a compensator of
        # the error, and the check that follows, 256 calibration rows through the result.
        ("compress_up", dict(kind="compress", N=14336, K=4096, r=32)),
    ]
    return [dict(c, name=n) for n, c in cases]


def _log(rng, lo, hi, step=1):
    """A size from lo to hi, evenly spread over its logarithm, in multiples of step."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return int(min(hi, max(lo, step * round(v / step))))


def draw(rng):
    kind = rng.choices(("decode", "rows", "moe_decode", "moe_rows", "pack", "compress"), (32, 26, 14, 14, 7, 7))[0]
    dtype = rng.choice(("fp16", "fp16", "bf16"))
    if kind in ("decode", "rows"):
        while True:
            M = _log(rng, 1, 16) if kind == "decode" else _log(rng, 17, 4096)
            N, K = _log(rng, 512, 14336, 16), _log(rng, 512, 14336, 64)
            if N * K <= 14336 * 4096 and M * N * K <= 4096 * 14336 * 4096:
                break
        r = rng.choice((0, 8, 16, 20, 24, 32, 48, 64, 128))
        int3 = dtype == "fp16" and N % 64 == 0 and 0 < r <= 64 and rng.random() < 0.5
        return _linear(M, N, K, r, dtype, rng.random() < 0.25, int3, rng.choice((1, 4, 8)) if kind == "decode" else 1)
    if kind in ("moe_decode", "moe_rows"):
        while True:
            T = _log(rng, 1, 64) if kind == "moe_decode" else _log(rng, 65, 4096)
            H, F = _log(rng, 512, 4096, 64), _log(rng, 512, 14336, 64)
            E = rng.choice((8, 16, 32, 64))
            topk, shared = rng.randint(1, 6), rng.choice((0, 0, 1, 2))
            # no more weights than the Mixtral-shaped layer, no more work than the 4096-token one
            if (E + shared) * H * F <= 8 * 4096 * 14336 and T * (topk + shared) * H * F <= 4096 * 8 * 2048 * 1408:
                break
        return _moe(T, H, F, E, topk, rng.choice(("0,8,16", "8", "16,32,64", "24,40")), shared,
                    rng.choice((32, 128)) if shared else 0, rng.choice((0.0, 1.2)), dtype)
    if kind == "pack":
        return dict(kind="pack", N=_log(rng, 512, 14336, 16), K=_log(rng, 512, 4096, 64), symmetric=rng.random() < 0.5)
    return dict(kind="compress", N=_log(rng, 512, 14336, 16), K=_log(rng, 512, 4096, 64), r=rng.choice((8, 16, 24, 32, 48)))


# ---------------------------------------------------------------- inputs

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)


def _type(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float16


def _weight(g, N, K, r, dt, symmetric=False, int3=False):
    """A packed weight of the distribution workloads.py uses, with a compensator of the size a fit to the
    quantization error gives: that error is about 0.2 sigma per element, so its leading singular values
    are about 0.2 sigma (sqrt(N) + sqrt(K)), and U and V share each one evenly."""
    pw = api.pack_w3(_normal(g, N, K).mul_(wl.WEIGHT_STD), symmetric=symmetric)
    if r == 0:
        return pw
    root = math.sqrt(0.2 * wl.WEIGHT_STD * (math.sqrt(N) + math.sqrt(K)))
    U, V = _normal(g, N, r).mul_(root / math.sqrt(N)), _normal(g, r, K).mul_(root / math.sqrt(K))
    if int3:
        u3, v3 = api.pack_lr3(U, V)
        return pw.with_int3_compensator(u3, v3, r)
    return pw.with_compensator(U.to(dt), V.to(dt))


def _routing(case, g):
    """Router outputs as in workloads.moe_routing: softmax, top-k, renormalised without shared experts."""
    T, E = case["T"], case["E"]
    logits = _normal(g, T, E)
    if case["zipf"] > 0:
        rank = torch.randperm(E, generator=g, device="cuda")
        logits = logits - case["zipf"] * torch.log(rank + 1.0)
    gates, ids = torch.softmax(logits, dim=1).topk(case["topk"], dim=1)
    if case["shared"]:
        sid = torch.arange(E, E + case["shared"], device="cuda").expand(T, -1)
        ids, gates = torch.cat([ids, sid], dim=1), torch.cat([gates, torch.ones_like(sid, dtype=gates.dtype)], dim=1)
    else:
        gates = gates / gates.sum(dim=1, keepdim=True)
    return ids.to(torch.int32).contiguous(), gates.to(torch.float32).contiguous()


def _spectrum_weight(g, N, K):
    """A weight with a few dominant directions over a flat bulk, as workloads.gen_weight_lowrank."""
    W = _normal(g, N, K).mul_(wl.WEIGHT_STD)
    a, b = _normal(g, N, 8), _normal(g, 8, K)
    a, b = a / a.norm(dim=0, keepdim=True), b / b.norm(dim=1, keepdim=True)
    gain = 6.0 * 0.75 ** torch.arange(8, device="cuda") * wl.WEIGHT_STD * (math.sqrt(N) + math.sqrt(K))
    return W.addmm_(a * gain, b).contiguous()


def prepare(case, seed):
    g = _generator(seed)
    kind = case["kind"]
    if kind == "linear":
        M, N, K, dt = case["M"], case["N"], case["K"], _type(case)
        return dict(kind=kind, X=_normal(g, M, K).to(dt),
                    weights=[_weight(g, N, K, case["r"], dt, case["symmetric"], case["int3"]) for _ in range(case["layers"])],
                    outs=[torch.empty((M, N), dtype=dt, device="cuda") for _ in range(case["layers"])],
                    workspace=api.new_workspace(api.gemm_workspace_bytes(M, N, K, case["r"])))
    if kind == "moe":
        H, F, E, dt = case["H"], case["F"], case["E"], _type(case)
        choices = [int(x) for x in case["ranks"].split(",")]
        pick = torch.randint(len(choices), (E,), generator=g, device="cuda").tolist()
        ranks = [choices[i] for i in pick] + [case["shared_rank"]] * case["shared"]
        experts = [tuple(_weight(g, n, k, r, dt) for n, k in ((F, H), (F, H), (H, F))) for r in ranks]
        ids, gates = _routing(case, g)
        return dict(kind=kind, layer=api.MoELayer(experts, H, F, bf16=dt == torch.bfloat16),
                    X=_normal(g, case["T"], H).to(dt), ids=ids, gates=gates)
    if kind == "pack":
        return dict(kind=kind, W=_normal(g, case["N"], case["K"]).mul_(wl.WEIGHT_STD), symmetric=case["symmetric"])
    return dict(kind=kind, W=_spectrum_weight(g, case["N"], case["K"]), r=case["r"],
                X=_normal(g, CALIBRATION_ROWS, case["K"]).to(torch.float16))


def run(state):
    kind = state["kind"]
    if kind == "linear":
        X, ws = state["X"], state["workspace"]
        return [api.w3lr_gemm(X, pw, out=out, workspace=ws) for pw, out in zip(state["weights"], state["outs"])]
    if kind == "moe":
        return state["layer"].forward(state["X"], state["ids"], state["gates"])
    if kind == "pack":
        return api.pack_w3(state["W"], symmetric=state["symmetric"]).q3
    # One outer iteration: from the second on, codes that fall on the other side of a rounding boundary
    # feed back, and two correct orders of summation drift apart.  U and V themselves are only defined up to
    # the signs (and, where singular values are close, a rotation) of their columns; what they do to
    # activations is not.
    pw, U, V, eps = api.compress_w3lr(state["W"], state["r"], iters=1)
    Y = api.w3lr_gemm(state["X"], pw.with_compensator(U.to(torch.float16), V.to(torch.float16)))
    return dict(q3=pw.q3, Y=Y, eps=torch.tensor(eps, dtype=torch.float64))


# ---------------------------------------------------------------- what a pass cannot do without

def _used(case):
    """Routed experts that receive a token, on average, for evenly spread tokens."""
    E, topk, T = case["E"], case["topk"], case["T"]
    return E * (1.0 - (1.0 - topk / E) ** T) + case["shared"]


def work(case):
    kind = case["kind"]
    if kind == "linear":
        M, N, K, r, layers = (case[k] for k in ("M", "N", "K", "r", "layers"))
        lr_bits = GROUP_BITS if case["int3"] else 16
        weight = N * K * GROUP_BITS / 8 + r * (N + K) * lr_bits / 8
        return {"bytes": layers * (weight + 2 * M * N) + 2 * M * K, "flops": layers * 2.0 * M * (N * K + r * (N + K))}
    if kind == "moe":
        T, H, F = case["T"], case["H"], case["F"]
        choices = [int(x) for x in case["ranks"].split(",")]
        rank = sum(choices) / len(choices)
        routed, shared = _used(case) - case["shared"], case["shared"]
        weights = 3 * ((routed + shared) * H * F * GROUP_BITS / 8 + 2 * (routed * rank + shared * case["shared_rank"]) * (H + F))
        flops = 2.0 * T * 3 * ((case["topk"] + shared) * H * F + (case["topk"] * rank + shared * case["shared_rank"]) * (H + F))
        return {"bytes": weights + 4 * T * H + 8 * T * (case["topk"] + shared), "flops": flops}
    N, K = case["N"], case["K"]
    if kind == "pack":
        return {"bytes": N * K * (4 + GROUP_BITS / 8), "flops": 8.0 * N * K}
    r, M = case["r"], CALIBRATION_ROWS
    # U V subtracted twice (error, stored target), three rounds of the two products of the subspace
    # iteration, 20 zero-point updates of about ten operations per weight, and the calibration rows
    return {"bytes": N * K * (4 + GROUP_BITS / 8) + 2 * M * (N + K), "flops": N * K * (16.0 * r + 200.0 + 2.0 * M)}


def tolerance(case):
    kind = case["kind"]
    if kind == "pack":
        return "exact"
    if kind == "compress":
        # codes and fp16 zero-points that sit on a rounding boundary go either way; one code is a few
        # percent of an output of the calibration rows
        return {"rel": 2e-3, "max": 0.2, "differ": 1e-3}
    # every dequantized weight and the output carry one rounding to 16 bits; an MoE layer has a second
    # linear, the 16-bit SwiGLU output and the 16-bit expert outputs on top
    if case["dtype"] == "bf16":
        return {"rel": 1e-2 if kind == "moe" else 6e-3}
    return {"rel": 2e-3 if kind == "moe" else 1e-3}
