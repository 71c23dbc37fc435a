"""Measured cases of the BASE-layer path: what a training or serving program
has this package do, call by call.

A training step scores its tokens against the expert embeddings (affinity),
solves the balanced assignment (assign, assign_batched), routes the token rows
into expert order (permute_batched), and after the experts runs the gated
residual and its gradient (gate_combine, gate_backward). A serving step routes
greedily (greedy_assign, permute, gate_combine). Each case makes one or a few
of these calls through the package's public functions, on synthetic inputs of
the layer's distributions: expert embeddings N(0, 1/d) and unit-variance
tokens, so scores are of unit variance; or tokens clustered around 8 experts,
where the assignment is contested. The solver cases take the scores as input,
so that a solve is compared on exactly the same scores.

Sizes are the package's workloads (T tokens, E experts, model dimension d) and
the ranges around them.
"""
from __future__ import annotations

import torch

import paper_2103_16716_amd as pb

DEV = "cuda"
KINDS = ("affinity", "assign", "batch", "infer", "gate")


def listed():
    return [
        # Scores of one training batch: 32768 tokens, 128 experts.
        dict(name="affinity-train", kind="affinity", T=32768, E=128, d=2048, dtype="bf16",
             gather=False),
        # The widest layer: twice the tokens, experts and width.
        dict(name="affinity-large", kind="affinity", T=65536, E=256, d=4096, dtype="bf16",
             gather=False),
        # A layer trained in fp32.
        dict(name="affinity-f32", kind="affinity", T=8192, E=64, d=1024, dtype="f32",
             gather=False),
        # Shuffled tokens read through the index, sizes that fill no tile.
        dict(name="affinity-ragged", kind="affinity", T=6000, E=100, d=1000, dtype="bf16",
             gather=True),
        # The smallest solve: a debug-size layer, where launches count.
        dict(name="assign-small", kind="assign", T=512, E=8, dist="normal", dtype="f32",
             warm=False),
        # One worker's problem of the paper's runs: 2 x 1024 tokens, 128 experts.
        dict(name="assign-worker", kind="assign", T=2048, E=128, dist="normal", dtype="f32",
             warm=False),
        # The exact integer variant on quantised scores.
        dict(name="assign-int16", kind="assign", T=4096, E=16, dist="normal", dtype="i16",
             warm=False),
        # A large training batch whose tokens crowd around 8 experts.
        dict(name="assign-train", kind="assign", T=32768, E=128, dist="mixture8", dtype="f32",
             warm=False),
        # The largest single solve.
        dict(name="assign-large", kind="assign", T=65536, E=256, dist="normal", dtype="f32",
             warm=False),
        # 256 workers' batches on one device: solve, then route the shuffled
        # rows to the experts and back.
        dict(name="batch-shuffled", kind="batch", B=256, T=2048, E=128, d=2048, dtype="bf16"),
        # A serving step around the experts: greedy routing, rows to the
        # experts, gated residual back in token order.
        dict(name="infer", kind="infer", T=8192, E=64, d=1024, dtype="bf16"),
        # A training step around the experts: gated residual and its gradient.
        dict(name="gate-train", kind="gate", T=32768, E=128, d=2048, dtype="bf16"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(KINDS)
    if kind == "affinity":
        return dict(kind=kind, T=_log_int(rng, 256, 65536), E=_log_int(rng, 8, 256),
                    d=8 * _log_int(rng, 16, 512) if rng.random() < 0.5 else
                    64 * _log_int(rng, 2, 64),
                    dtype="f32" if rng.random() < 0.25 else "bf16", gather=rng.random() < 0.4)
    if kind == "assign":
        E = _log_int(rng, 8, 256)
        C = _log_int(rng, 8, min(512, 65536 // E))
        i16 = rng.random() < 0.25
        if i16:   # exact solves: the range of the integer workload
            E, C = min(E, 32), min(C, 256)
        return dict(kind=kind, T=E * C, E=E, dtype="i16" if i16 else "f32",
                    dist="normal" if i16 else rng.choice(("normal", "mixture8")),
                    warm=not i16 and rng.random() < 0.3)
    if kind == "batch":
        E = 4 * _log_int(rng, 2, 32)
        C = _log_int(rng, 4, 2048 // E)
        return dict(kind=kind, B=_log_int(rng, 2, 256), T=E * C, E=E,
                    d=8 * _log_int(rng, 16, 256), dtype="bf16")
    E = _log_int(rng, 8, 256)
    dtype = "f32" if rng.random() < 0.25 else "bf16"
    if kind == "infer":   # any number of tokens
        return dict(kind=kind, T=_log_int(rng, 64, 32768), E=E, d=8 * _log_int(rng, 16, 512),
                    dtype=dtype)
    C = _log_int(rng, 8, min(1024, 32768 // E))   # the balanced routing of training
    return dict(kind=kind, T=E * C, E=E, d=8 * _log_int(rng, 16, 256), dtype=dtype)


# ------------------------------------------------------------------ inputs --

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) + 2103_16716)
    return g


def _randn(shape, g, dtype, scale=1.0):
    """N(0, scale^2), drawn in fp32 and rounded to the storage type."""
    x = torch.randn(shape, generator=g, device=DEV, dtype=torch.float32)
    if scale != 1.0:
        x *= scale
    return x.to(torch.bfloat16) if dtype == "bf16" else x


def _scores(n, E, g, dist="normal"):
    """Scores h_t . w_e of unit-variance tokens; "mixture8": of tokens
    h = w_c + 0.3 z around 8 of the experts (|w_c| = 1, the other embeddings
    nearly orthogonal at d = 2048)."""
    S = torch.randn((n, E), generator=g, device=DEV, dtype=torch.float32)
    if dist == "normal":
        return S
    k = min(8, E)
    near = torch.randn((E, E), generator=g, device=DEV, dtype=torch.float32) / 2048 ** 0.5
    near.fill_diagonal_(1.0)
    centres = torch.randperm(E, generator=g, device=DEV)[:k]
    c = centres[torch.randint(0, k, (n,), generator=g, device=DEV)]
    return S.mul_(0.3).add_(near[c])


def _balanced_routing(T, E, g):
    """A balanced assignment and its stable sort vector."""
    a = (torch.randperm(T, generator=g, device=DEV) % E).to(torch.int32)
    return a, torch.sort(a, stable=True).indices.to(torch.int32)


def prepare(case, seed):
    g = _gen(seed)
    kind, T, E = case["kind"], case["T"], case["E"]
    if kind == "affinity":
        d, dt = case["d"], case["dtype"]
        rows = None
        if case["gather"]:
            rows = torch.randperm(T, generator=g, device=DEV).to(torch.int32)
        return dict(kind=kind, W=_randn((E, d), g, dt, d ** -0.5), H=_randn((T, d), g, dt),
                    rows=rows)
    if kind == "assign":
        st = dict(kind=kind, prices=None,
                  ws=torch.empty(pb.assign_workspace_size(T, E), dtype=torch.uint8, device=DEV))
        S = _scores(T, E, g, case["dist"])
        if case["dtype"] == "i16":   # about 15 bits of the score range
            S = (S * 4096.0).round_().clamp_(-32767, 32767).to(torch.int16)
        if case["warm"]:   # the next batch's solve starts from this batch's prices
            st["prices"] = pb.assign(S, workspace=st["ws"]).prices
            S = S + 0.05 * torch.randn(S.shape, generator=g, device=DEV)
        st["S"] = S
        return st
    if kind == "batch":
        B, d = case["B"], case["d"]
        return dict(kind=kind, S=_scores(B * T, E, g).view(B, T, E),
                    H=_randn((B * T, d), g, case["dtype"]),
                    shuffle=torch.randperm(B * T, generator=g, device=DEV).to(torch.int32),
                    ws=torch.empty(pb.assign_batched_workspace_size(B, T, E), dtype=torch.uint8,
                                   device=DEV))
    d, dt = case["d"], case["dtype"]
    st = dict(kind=kind, S=_scores(T, E, g), H=_randn((T, d), g, dt), F=_randn((T, d), g, dt))
    if kind == "infer":
        n = int(pb.lib().base_greedy_workspace_size(T, E))
        st["ws"] = torch.empty(max(n, 256), dtype=torch.uint8, device=DEV)
        return st
    st["assign"], st["perm"] = _balanced_routing(T, E, g)
    st["offsets"] = pb.balanced_offsets(T, E, DEV)
    st["W"] = _randn((E, d), g, dt, d ** -0.5)
    st["dY"] = _randn((T, d), g, dt)
    return st


# -------------------------------------------------------------------- pass --

def run(st):
    kind = st["kind"]
    if kind == "affinity":
        return pb.affinity(st["H"], st["W"], rows=st["rows"])
    if kind == "assign":
        if st["prices"] is None:
            r = pb.assign(st["S"], workspace=st["ws"], sync_stats=False)
        else:
            r = pb.assign(st["S"], workspace=st["ws"], sync_stats=False, warm_start=True,
                          out_prices=st["prices"].clone())
        return dict(assign=r.assign, perm=r.perm, prices=r.prices)
    if kind == "batch":
        r = pb.assign_batched(st["S"], workspace=st["ws"], sync_stats=False)
        X = pb.permute_batched(st["H"], r.perm, shuffle=st["shuffle"])
        Y = pb.permute_batched(X, r.perm, shuffle=st["shuffle"], inverse=True)
        return dict(assign=r.assign, perm=r.perm, prices=r.prices, X=X, Y=Y)
    S, H, F = st["S"], st["H"], st["F"]
    if kind == "infer":
        a, perm, offsets = pb.greedy_assign(S, workspace=st["ws"])
        X = pb.permute(H, perm)
        return dict(assign=a, perm=perm, offsets=offsets, X=X,
                    Y=pb.gate_combine(F, H, S, a, perm))
    Y = pb.gate_combine(F, H, S, st["assign"], st["perm"])
    dH, dF, dW, dS = pb.gate_backward(st["dY"], F, H, st["W"], S, st["assign"], st["perm"],
                                      offsets=st["offsets"])
    return dict(Y=Y, dH=dH, dF=dF, dW=dW, dS=dS)


# ------------------------------------------------------- work and accuracy --

def work(case):
    kind, T, E = case["kind"], case["T"], case["E"]
    sz = {"bf16": 2, "f32": 4, "i16": 2}[case["dtype"]]
    if kind == "affinity":
        d = case["d"]
        return dict(bytes=(T + E) * d * sz + 4 * T * E + (4 * T if case["gather"] else 0),
                    flops=2 * T * E * d)
    if kind == "assign":   # every score once; assign, perm and prices out
        return dict(bytes=sz * T * E + 8 * T + (8 if sz == 2 else 4) * E, flops=T * E)
    if kind == "batch":    # the solves, then the rows to the experts and back
        N, d = case["B"] * T, case["d"]
        return dict(bytes=4 * N * E + 8 * N + 4 * case["B"] * E + 4 * N + 4 * N * d * sz,
                    flops=N * E)
    d = case["d"]
    if kind == "infer":    # scores, H and F in; X and Y out
        return dict(bytes=4 * T * E + 8 * T + 4 * T * d * sz, flops=T * E + 2 * T * d)
    # gate: F, H, dY and W in; Y, dH, dF, dW, dS out; a score per token
    return dict(bytes=6 * T * d * sz + E * d * (sz + 4) + 16 * T, flops=10 * T * d)


def tolerance(case):
    kind = case["kind"]
    if kind == "affinity":
        # fp32 sums of d products (exact products for bf16 inputs): against
        # 64 bits the relative 2-norm error is 1e-7 to 6e-7 over the range.
        return {"rel": 3e-6, "max": 3e-5}
    if kind in ("assign", "batch"):
        # The solver is deterministic whatever the route or the batch, and
        # rows are moved bit for bit.
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 3e-6, "max": 3e-5}
    # One rounding to bf16 of each stored value (relative 2-norm error
    # 1.7e-3, at most half a unit in the last place: 3.9e-3).
    return {"rel": 7e-3, "max": 1.6e-2}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("assign", "batch"):
        return None   # any assignment within T * eps of the optimum is a right one
    st = prepare(case, seed)
    if kind == "affinity":
        W = st["W"].double().t().contiguous()
        S = torch.empty((case["T"], case["E"]), dtype=torch.float64, device=DEV)
        for t0 in range(0, case["T"], 8192):
            sel = slice(t0, t0 + 8192)
            h = st["H"][sel] if st["rows"] is None else st["H"][st["rows"][sel].long()]
            S[sel] = h.double() @ W
        return S
    S, H, F = st["S"].double(), st["H"].double(), st["F"].double()
    if kind == "infer":
        a = st["S"].argmax(dim=1)
        perm = torch.sort(a, stable=True).indices
        Y = H.clone()
        Y[perm] += torch.sigmoid(S[perm, a[perm]])[:, None] * F
        return dict(assign=None, perm=None, offsets=None, X=H[perm], Y=Y)
    a, perm = st["assign"].long(), st["perm"].long()
    W, dY = st["W"].double(), st["dY"].double()
    f = torch.empty_like(F)
    f[perm] = F
    g = torch.sigmoid(S.gather(1, a[:, None]))
    dS = (g * (1 - g)).squeeze(1) * (dY * f).sum(dim=1)
    dW = torch.zeros_like(W).index_add_(0, a, dS[:, None] * H)
    return dict(Y=g * f + H, dH=dY + dS[:, None] * W[a], dF=(g * dY)[perm], dW=dW, dS=dS)
