"""The work a user of this package gives it, as cases to be measured: fused steps from one decode row to a
16K-token prefill, the token split, GEMMs of both weight layouts, the overlapped pair, one layer boundary under
the per-iteration policy, and trains of boundaries as an engine runs them, in decode and in prefill.

A case is a dict of plain values:
  kind    fused | split | gemm | overlap | layer | train
  fused, split, overlap   N rows, H hidden size, P partials, budget (cu_budget)
  gemm, overlap           M, K, Nout, layout ("nk" or "kn")
  layer, train            T tokens, H, P, K1 and N2 of the boundary (layer), layers (train)
Sizes are those of the workload configurations and of the benchmark (70B-class: H = 8192, P = 8; 8B-class:
H = 4096, P = 2), or lie between them.

All calls go through the package's public functions with outputs allocated beforehand, as a serving loop has
them; inputs are bf16 with the distributions of the workload configurations.
"""
import math

import torch

import paper_2505_11329_amd as tw

DEV = "cuda:0"
# G1's depth K1 and G2's width N2 of the two boundaries of a 70B-class layer at TP = 8
ATTENTION, MLP = (1024, 3584), (3584, 1280)
TRAIN_SPLIT_THRESHOLD = 3072  # TW_TRAIN_SPLIT_THRESHOLD of tw.h

_second_stream = []


def second_stream():
    """A stream whose kernels run side by side with the current stream's; a program sets it up once."""
    if not _second_stream:
        here = torch.cuda.current_stream()
        for _ in range(16):
            s = torch.cuda.Stream()
            if tw.streams_overlap(here, s):
                break
        _second_stream.append(s)
    return _second_stream[0]


def third_stream():
    """Another one that runs side by side with the second."""
    second = second_stream()
    if len(_second_stream) < 2:
        for _ in range(16):
            s = torch.cuda.Stream()
            if tw.streams_overlap(second, s):
                break
        _second_stream.append(s)
    return _second_stream[1]


def listed():
    return [
        # one decode iteration's fused step: a few rows, launch and latency are everything
        dict(name="fused_decode", kind="fused", N=16, H=8192, P=8, budget=0),
        # 8B-class chunk at TP = 2
        dict(name="fused_8b_tp2", kind="fused", N=2048, H=4096, P=2, budget=0),
        # one GPU's share of an 8K-token 70B-class batch, confined to 32 compute units (the headline setting)
        dict(name="fused_70b_budget32", kind="fused", N=1024, H=8192, P=8, budget=32),
        # a token count and a number of partials that are no powers of two, another hidden size
        dict(name="fused_ragged", kind="fused", N=1531, H=5120, P=6, budget=0),
        # long prefill: beyond every cache
        dict(name="fused_prefill", kind="fused", N=16384, H=8192, P=4, budget=0),
        # the token split on two streams, each half confined to 64 compute units
        dict(name="split_4k", kind="split", N=4096, H=8192, P=4, budget=64),
        # the projection of the overlap demonstration, on its own
        dict(name="gemm_demo", kind="gemm", M=2048, K=8192, Nout=3584, layout="nk"),
        # weights stored [K x N], odd sizes
        dict(name="gemm_kn_ragged", kind="gemm", M=3001, K=4104, Nout=4096, layout="kn"),
        # the fused step of one half beside the projection of the other half
        dict(name="overlap_demo", kind="overlap", N=2048, H=8192, P=8, budget=tw.CU_SHARED, M=2048, K=8192, Nout=3584,
             layout="nk"),
        # one boundary of an iteration with a few hundred tokens: small prefill or a large decode batch
        dict(name="layer_small", kind="layer", T=333, H=8192, P=8, K1=1024, N2=3584),
        # decode iteration: eight boundaries (four 70B-class layers) of 16 tokens, weights from memory
        dict(name="train_decode", kind="train", T=16, H=8192, P=8, layers=8),
        # prefill iteration: the same of 8192 tokens, woven in two splits
        dict(name="train_prefill", kind="train", T=8192, H=8192, P=8, layers=8),
    ]


def draw(rng):
    def spread(lo, hi, multiple=1):
        v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        return max(multiple, int(v / multiple + 0.5) * multiple)

    def partials():
        return rng.choice((1, 2, 2, 3, 4, 4, 6, 8, 8, 8, 12, 16))

    def hidden():
        return rng.choice((2048, 4096, 4096, 5120, 8192, 8192, spread(512, 16384, 8)))

    kind = rng.choice(("fused", "fused", "split", "gemm", "gemm", "overlap", "layer", "layer", "train"))
    if kind == "fused":
        return dict(kind=kind, N=spread(1, 16384), H=hidden(), P=partials(),
                    budget=rng.choice((0, 0, 0, 0, 16, 32, 64, tw.CU_SHARED)))
    if kind == "split":
        return dict(kind=kind, N=spread(128, 16384), H=hidden(), P=partials(), budget=rng.choice((0, 16, 32, 64)))
    if kind == "gemm":
        return dict(kind=kind, M=spread(1, 8192), K=spread(256, 8192, 8), Nout=spread(256, 8192, 8),
                    layout=rng.choice(("nk", "nk", "kn")))
    if kind == "overlap":
        return dict(kind=kind, N=spread(128, 4096), H=hidden(), P=partials(), budget=rng.choice((32, 64, tw.CU_SHARED)),
                    M=spread(128, 4096), K=spread(1024, 8192, 8), Nout=spread(1024, 8192, 8),
                    layout=rng.choice(("nk", "nk", "kn")))
    if kind == "layer":
        H, P = rng.choice(((8192, 8), (8192, 8), (8192, 4), (4096, 2), (4096, 4)))
        K1, N2 = rng.choice((ATTENTION, MLP, (spread(512, 4096, 64), spread(1024, 4096, 64))))
        return dict(kind=kind, T=spread(1, 8192), H=H, P=P, K1=K1, N2=N2)
    return dict(kind=kind, T=spread(1, 8192), H=8192, P=8, layers=rng.choice((2, 4, 6)))


# ---- inputs ---------------------------------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal(g, shape, std):
    return torch.empty(shape, dtype=torch.bfloat16, device=DEV).normal_(0.0, std, generator=g)


def _norm_weight(g, H):
    return torch.empty((H,), dtype=torch.bfloat16, device=DEV).uniform_(0.5, 1.5, generator=g)


def _fused_inputs(g, N, H, P):
    """Partials of smaller variance than the residual stream, whose outliers are 1 % of its entries."""
    residual = _normal(g, (N, H), 1.0)
    outlier = torch.empty((N, H), dtype=torch.bfloat16, device=DEV).uniform_(generator=g) < 0.01
    residual = torch.where(outlier, residual * 50, residual)
    return dict(partials=[_normal(g, (N, H), 0.25 if P > 4 else 0.5) for _ in range(P)], residual=residual,
                weight=_norm_weight(g, H), eps=1e-5, out=torch.empty_like(residual),
                residual_out=torch.empty_like(residual))


def _gemm_inputs(g, case):
    M, K, N = case["M"], case["K"], case["Nout"]
    nk = case["layout"] == "nk"
    return dict(A=_normal(g, (M, K), 0.02), B=_normal(g, (N, K) if nk else (K, N), 0.02),
                C=torch.empty((M, N), dtype=torch.bfloat16, device=DEV), b_layout=tw.B_NK if nk else tw.B_KN)


def _boundary(g, T, H, K1, N2, fused):
    return dict(fused, X1=_normal(g, (T, K1), 1.0), W1=_normal(g, (H, K1), 0.02), W2=_normal(g, (N2, H), 0.02),
                Y=torch.empty((T, N2), dtype=torch.bfloat16, device=DEV))


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    s = dict(case=case)
    if kind in ("fused", "split", "overlap"):
        s["fused"] = dict(_fused_inputs(g, case["N"], case["H"], case["P"]), cu_budget=case["budget"])
    if kind in ("gemm", "overlap"):
        s["gemm"] = _gemm_inputs(g, case)
    if kind == "split":
        s["row"] = tw.split_point(case["N"], 128)
        s["streams"] = (second_stream(), third_stream())
    if kind == "overlap":
        s["streams"] = (second_stream(), torch.cuda.current_stream())
    if kind in ("layer", "train"):
        T, H, P = case["T"], case["H"], case["P"]
        s["streams"] = (torch.cuda.current_stream(), second_stream())
        first = _fused_inputs(g, T, H, P)
        if kind == "layer":
            s["boundary"] = _boundary(g, T, H, case["K1"], case["N2"], first)
        else:
            # the residual stream runs through the boundaries; the partials of the other ranks lie in the
            # communication buffers that every boundary uses; weights are each boundary's own
            s["boundaries"] = []
            residual = first["residual"]
            for i in range(case["layers"]):
                fused = dict(partials=first["partials"], residual=residual, weight=_norm_weight(g, H), eps=1e-5,
                             out=torch.empty_like(residual), residual_out=torch.empty_like(residual))
                residual = fused["residual_out"]
                s["boundaries"].append(_boundary(g, T, H, *(MLP if i % 2 else ATTENTION), fused))
            s["row"] = T
            if T >= TRAIN_SPLIT_THRESHOLD:
                (K1, N2), cus = ATTENTION, tw.device_cu_count()
                s["row"] = tw.smart_split_point(T, 64, [H, N2], cus, gemm_k=[K1, H])[0]
    return s


# ---- one pass -------------------------------------------------------------------------------------------------

def run(state):
    kind = state["case"]["kind"]
    if kind == "fused":
        return tw.reduce_add_rmsnorm(**state["fused"])
    if kind == "split":
        a, b = state["streams"]
        return tw.split_launch(split_row=state["row"], stream_a=a, stream_b=b, **state["fused"])
    if kind == "gemm":
        return tw.gemm_bf16(**state["gemm"])
    if kind == "overlap":
        return tw.overlap_launch(state["fused"], state["gemm"], *state["streams"])
    compute, comm = state["streams"]
    if kind == "layer":
        out, residual_out, Y, _ = tw.weave_layer_auto(stream_compute=compute, stream_comm=comm, **state["boundary"])
        return out, residual_out, Y
    tw.weave_train(state["boundaries"], state["row"], compute, comm)
    return [(b["out"], b["residual_out"], b["Y"]) for b in state["boundaries"]]


# ---- what a pass cannot do without, and how exact it is ---------------------------------------------------------

def _fused_work(N, H, P):
    return dict(bytes=(P + 3) * N * H * 2 + H * 2, flops=(P + 6) * N * H)


def _gemm_work(M, N, K):
    return dict(bytes=2 * (M * K + N * K + M * N), flops=2 * M * N * K)


def _boundary_work(T, H, P, K1, N2):
    # G1's result and the fused step's output pass through memory between the kernels, but a boundary has to read
    # only what comes from outside (X1, W1, the other P - 1 partials, the residual, W2) and to write what it is
    # asked for (out, residual_out, Y)
    return dict(bytes=2 * (T * K1 + H * K1 + (P - 1 + 1 + 2) * T * H + H + N2 * H + T * N2),
                flops=2 * T * H * (K1 + N2) + (P + 6) * T * H)


def work(case):
    kind = case["kind"]
    parts = []
    if kind in ("fused", "split", "overlap"):
        parts.append(_fused_work(case["N"], case["H"], case["P"]))
    if kind in ("gemm", "overlap"):
        parts.append(_gemm_work(case["M"], case["Nout"], case["K"]))
    if kind == "layer":
        parts.append(_boundary_work(case["T"], case["H"], case["P"], case["K1"], case["N2"]))
    if kind == "train":
        parts += [_boundary_work(case["T"], case["H"], case["P"], *(MLP if i % 2 else ATTENTION))
                  for i in range(case["layers"])]
    return dict(bytes=sum(p["bytes"] for p in parts), flops=sum(p["flops"] for p in parts))


def tolerance(case):
    # bf16 results of fp32 sums: another order of the additions moves a value across a rounding boundary now and
    # then, by one bf16 step (2^-8 of the value at most); where results pass through bf16 between kernels such
    # steps carry on through the next products
    if case["kind"] in ("layer", "train"):
        return dict(rel=5e-3, max=5e-2)
    return dict(rel=2e-3, max=1e-2)
