"""The work that programs have the FLARE++ library do, as timed cases.

A case names an operation, its sizes (batch B, tokens N, width C, heads H,
routes M), a storage type and the spread of the learned seeds:

  forward     the mixer forward (inference)
  flare       the fixed-query mixer forward (inference)
  train       the training pair: forward that keeps its statistics, backward
  backward    the stand-alone backward (activation recomputation)
  block       a training step of the pre-norm residual block
  primitives  project, then an encode and a decode routing call on their own

``seeds`` scales the seed initialisation N(0, 1 / D): 1 is a fresh model, 4 a
trained one whose routes have become selective.
"""

from __future__ import annotations

import math

import torch

from paper_2608_11519_amd import flarepp as fp

EPS = 1e-5
WEIGHTS = ("Wk", "Wv", "Wkt", "Wvt", "Wo")


def _case(op, dtype, B, N, C, H, M, seeds, x="normal", name=None):
    c = dict(op=op, dtype=dtype, B=B, N=N, C=C, H=H, M=M, seeds=seeds, x=x)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # a small mesh in single precision: the latency of one call
        _case("forward", "f32", 1, 1024, 64, 4, 32, 1.0, name="forward small f32"),
        # two ragged clouds of under a thousand points: launches and host work
        _case("forward", "bf16", 2, 777, 128, 8, 64, 4.0, name="forward ragged"),
        # a batch of 128 x 128 grids (structured PDE problems)
        _case("forward", "bf16", 4, 16384, 128, 8, 128, 1.0, name="forward grid2d"),
        # irregular meshes with Fourier features, the wide model
        _case("forward", "bf16", 2, 50000, 256, 8, 256, 1.0, "fourier", name="forward mesh"),
        # a million tokens on one GPU
        _case("forward", "bf16", 1, 1 << 20, 128, 8, 512, 1.0, name="forward mesh3d"),
        # the fixed-query baseline on long sequences of embedded symbols
        _case("flare", "bf16", 32, 4096, 128, 8, 64, 1.0, "embedding", name="flare lra"),
        # a training step of the residual block on the same sequences
        _case("block", "bf16", 32, 4096, 128, 8, 64, 4.0, "embedding", name="block step lra"),
        # training on the grids
        _case("train", "bf16", 4, 16384, 128, 8, 128, 4.0, name="train grid2d"),
        # training on the irregular meshes, the wide model
        _case("train", "bf16", 2, 50000, 256, 8, 256, 4.0, "fourier", name="train mesh"),
        # the million-token backward with the forward recomputed
        _case("backward", "bf16", 1, 1 << 20, 128, 8, 512, 4.0, name="backward mesh3d"),
        # single-precision training on a ragged cloud (PDE solvers)
        _case("train", "f32", 1, 20011, 64, 4, 100, 4.0, name="train f32"),
        # the routing calls on their own at a width without a fused path
        _case("primitives", "bf16", 3, 9973, 96, 3, 200, 4.0, name="primitives c96"),
    ]


def draw(rng):
    """Another case of the same ranges: 2^9 .. 2^20 tokens, 8 .. 512 routes,
    the widths and head widths of the listed ones and those between."""
    while True:
        op = rng.choice(["forward", "forward", "train", "train", "backward", "block", "flare", "primitives"])
        dtype = "f32" if rng.random() < 0.15 else "bf16"
        C = rng.choice([64, 96, 128, 128, 128, 256])
        D = rng.choice([d for d in (16, 16, 32, 64) if C % d == 0])
        tokens = 2.0 ** rng.uniform(9, 20)
        B = min(rng.choice([1, 1, 2, 3, 4, 8, 32]), max(1, int(tokens) // 128))
        N = max(64, int(tokens / B))
        M = int(round(2.0 ** rng.uniform(3, 9)))
        c = _case(op, dtype, B, N, C, C // D, M, rng.choice([1.0, 4.0]), rng.choice(["normal", "fourier", "embedding"]))
        # no dearer than the largest listed case: single precision has 1/16 of
        # the matrix rate, the paths without fusion move more
        cost = work(c)["flops"] * (16 if dtype == "f32" else 2)
        if cost <= work(listed()[9])["flops"]:
            return c


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _sizes(case):
    return tuple(case[k] for k in ("B", "N", "C", "H", "M"))


def _inputs(case, seed):
    """The tensors of a case in its storage type, from the seed alone."""
    B, N, C, H, M = _sizes(case)
    D, dt = C // H, _dtype(case)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)

    if case["x"] == "normal":
        X = normal(B, N, C)
    elif case["x"] == "fourier":  # random Fourier features of points in the plane, with noise
        pts = torch.rand((B, N, 2), generator=g, device="cuda")
        ang = 2 * math.pi * torch.matmul(pts, 4.0 * normal(2, C // 2))
        X = torch.cat([ang.cos(), ang.sin()], dim=-1) + math.sqrt(0.1) * normal(B, N, C)
    else:  # embedded symbols of an alphabet of 256
        X = normal(256, C)[torch.randint(0, 256, (B, N), generator=g, device="cuda")]
    t = {"X": X.to(dt)}
    a = math.sqrt(3.0 / C)
    for k in WEIGHTS:
        t[k] = ((2 * torch.rand((C, C), generator=g, device="cuda") - 1) * a).to(dt)
    t["seeds"] = (normal(H, M, D) * (case["seeds"] / math.sqrt(D))).to(dt)
    if case["op"] in ("train", "backward", "block"):
        t["dO"] = normal(B, N, C).to(dt)
    if case["op"] == "block":
        t["gamma"] = (1 + 0.1 * normal(C)).to(dt)
        t["beta"] = (0.1 * normal(C)).to(dt)
    if case["op"] == "primitives":
        t["q"] = normal(B, H, M, D) * (case["seeds"] / math.sqrt(D))
    return t


def prepare(case, seed):
    """Inputs, and the workspace that a program keeps between its steps."""
    B, N, C, H, M = _sizes(case)
    code = fp.F32 if case["dtype"] == "f32" else fp.BF16
    t = _inputs(case, seed)
    if case["op"] in ("train", "backward"):
        n = fp.flarepp_mixer_backward_workspace_bytes(code, B, N, C, H, M)
    elif case["op"] == "block":
        n = max(fp.flarepp_block_workspace_bytes(code, B, N, C, H, M),
                fp.flarepp_block_backward_workspace_bytes(code, B, N, C, H, M))
    elif case["op"] == "flare":
        n = fp.flarepp_flare_workspace_bytes(code, B, N, C, H, M)
    elif case["op"] == "primitives":
        n = max(fp.flarepp_project_workspace_bytes(code, C),
                fp.flarepp_route_workspace_bytes(fp.ENCODE, code, B, H, N, M, C // H),
                fp.flarepp_route_workspace_bytes(fp.DECODE, code, B, H, N, M, C // H))
    else:
        n = fp.flarepp_mixer_workspace_bytes(code, B, N, C, H, M)
    t["ws"] = torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")
    t["case"] = case
    return t


def run(s):
    op, H, ws = s["case"]["op"], s["case"]["H"], s["ws"]
    w = [s[k] for k in WEIGHTS]
    if op == "forward":
        return fp.flarepp_mixer_forward(s["X"], *w, s["seeds"], H=H, ws=ws)
    if op == "flare":
        return fp.flarepp_flare_forward(s["X"], s["Wk"], s["Wv"], s["Wo"], s["seeds"], H=H, ws=ws)
    if op == "train":
        O = fp.flarepp_mixer_forward_train(s["X"], *w, s["seeds"], H=H, ws=ws)
        return O, fp.flarepp_mixer_backward_from_saved(s["X"], *w, s["seeds"], s["dO"], H=H, ws=ws)
    if op == "backward":
        return fp.flarepp_mixer_backward(s["X"], *w, s["seeds"], s["dO"], H=H, ws=ws)
    if op == "block":
        O = fp.flarepp_block_forward(s["X"], s["gamma"], s["beta"], *w, s["seeds"], H=H, eps=EPS, ws=ws)
        return O, fp.flarepp_block_backward(s["X"], s["gamma"], s["beta"], *w, s["seeds"], s["dO"], H=H, eps=EPS, ws=ws)
    K, V, _, _ = fp.flarepp_project(s["X"], s["Wk"], s["Wv"], H=H, ws=ws)
    Z, lse = fp.flarepp_route(fp.ENCODE, s["q"], K, V, want_lse=True, ws=ws)
    Y = fp.flarepp_route(fp.DECODE, K, s["q"], Z, ws=ws)
    return K, V, Z, lse, Y


def work(case):
    """Bytes: every input read and every output written once.  Operations:
    per token 2 C^2 for a projection, 4 M C for a routing call, and for their
    gradients twice 2 C^2 and 10 M C (with the scores again)."""
    B, N, C, H, M = _sizes(case)
    T, es, op = B * N, 4 if case["dtype"] == "f32" else 2, case["op"]
    small = 5 * C * C + M * C
    if op == "forward":
        return {"bytes": es * (2 * T * C + small), "flops": T * (10 * C * C + 12 * M * C)}
    if op == "flare":
        return {"bytes": es * (2 * T * C + small), "flops": T * (6 * C * C + 8 * M * C)}
    if op == "primitives":
        return {"bytes": es * (4 * T * C + 2 * C * C) + 4 * B * M * (2 * C + H), "flops": T * (4 * C * C + 8 * M * C)}
    outs = (2 if op == "backward" else 3) * es * T * C + 4 * T * C
    flops = T * ((28 if op == "backward" else 30) * C * C + 42 * M * C)
    return {"bytes": outs + (es + 4) * small, "flops": flops}


def tolerance(case):
    """About four times the distance from the float64 results.  Single
    precision (exponentials, sums over tokens): 3e-7 to 1.8e-6.  bf16 (every
    product's operands are rounded): 1.7e-3 to 3.2e-3 for forward results,
    which pass through three routing calls, and up to 6.4e-3 for gradients,
    which pass through six."""
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    if case["op"] in ("forward", "flare", "primitives"):
        return {"rel": 1e-2, "max": 0.3}
    return {"rel": 2e-2, "max": 0.5}


# ---------------------------------------------------------------------------
# The same results in float64, by plain torch
# ---------------------------------------------------------------------------
def _step(B, H, M):
    return max(64, (1 << 26) // (B * H * M))


def _heads(A, H):
    B, N, C = A.shape
    return A.view(B, N, H, C // H).transpose(1, 2).contiguous()


def _merge(A):
    B, H, N, D = A.shape
    return A.transpose(1, 2).reshape(B, N, H * D)


def _T(A):
    return A.transpose(-1, -2).contiguous()


def _encode(q, K, V):
    """softmax over the tokens of q K^T / sqrt(D), times V; its log-normaliser."""
    B, H, N, D = K.shape
    q = q.expand(B, -1, -1, -1).contiguous()
    n, sc = _step(B, H, q.shape[2]), 1 / math.sqrt(D)
    L = torch.full(q.shape[:3], -math.inf, dtype=q.dtype, device=q.device)
    for a in range(0, N, n):
        L = torch.logaddexp(L, torch.logsumexp(torch.matmul(q, _T(K[:, :, a:a + n])) * sc, dim=-1))
    out = torch.zeros_like(q)
    for a in range(0, N, n):
        P = (torch.matmul(q, _T(K[:, :, a:a + n])) * sc - L[..., None]).exp_()
        out += torch.matmul(P, V[:, :, a:a + n].contiguous())
    return out, L


def _decode(K, q, Z):
    """Tokens read the routes: softmax over the routes of K q^T / sqrt(D), times Z."""
    B, H, N, D = K.shape
    q = q.expand(B, -1, -1, -1).contiguous()
    n, Y = _step(B, H, q.shape[2]), torch.empty_like(K)
    for a in range(0, N, n):
        P = torch.softmax(torch.matmul(K[:, :, a:a + n].contiguous(), _T(q)) / math.sqrt(D), dim=-1)
        Y[:, :, a:a + n] = torch.matmul(P, Z)
    return Y


def _encode_grad(q, K, V, out, L, dout):
    """Gradients of _encode with respect to q, K and V."""
    B, H, N, D = K.shape
    q = q.expand(B, -1, -1, -1).contiguous()
    n, sc = _step(B, H, q.shape[2]), 1 / math.sqrt(D)
    c = (dout * out).sum(-1, keepdim=True)
    dq, dK, dV = torch.zeros_like(q), torch.empty_like(K), torch.empty_like(V)
    for a in range(0, N, n):
        k = K[:, :, a:a + n].contiguous()
        P = (torch.matmul(q, _T(k)) * sc - L[..., None]).exp_()
        dV[:, :, a:a + n] = torch.matmul(_T(P), dout)
        dS = P.mul_(torch.matmul(dout, _T(V[:, :, a:a + n])).sub_(c)).mul_(sc)
        dK[:, :, a:a + n] = torch.matmul(_T(dS), q)
        dq += torch.matmul(dS, k)
    return dq, dK, dV


def _decode_grad(K, q, Z, Y, dY):
    """Gradients of _decode with respect to K, q and Z."""
    B, H, N, D = K.shape
    q = q.expand(B, -1, -1, -1).contiguous()
    n, sc = _step(B, H, q.shape[2]), 1 / math.sqrt(D)
    dK, dq, dZ = torch.empty_like(K), torch.zeros_like(q), torch.zeros_like(q)
    for a in range(0, N, n):
        k, dy = K[:, :, a:a + n].contiguous(), dY[:, :, a:a + n].contiguous()
        P = torch.softmax(torch.matmul(k, _T(q)) * sc, dim=-1)
        dZ += torch.matmul(_T(P), dy)
        dS = P.mul_(torch.matmul(dy, _T(Z)).sub_((dy * Y[:, :, a:a + n]).sum(-1, keepdim=True))).mul_(sc)
        dK[:, :, a:a + n] = torch.matmul(dS, q)
        dq += torch.matmul(_T(dS), k)
    return dK, dq, dZ


def _mixer(X, t, H):
    """(O, what the gradient needs) of the mixer."""
    K, V, Kt, Vt = (_heads(torch.matmul(X, t[k]), H) for k in ("Wk", "Wv", "Wkt", "Wvt"))
    Q, L1 = _encode(t["seeds"][None], Kt, Vt)
    Z, L2 = _encode(Q, K, V)
    Y = _decode(K, Q, Z)
    return torch.matmul(_merge(Y), t["Wo"]), (K, V, Kt, Vt, Q, L1, Z, L2, Y)


def _mixer_grad(X, t, H, kept, dO):
    K, V, Kt, Vt, Q, L1, Z, L2, Y = kept
    B, N, C = X.shape
    dY = _heads(torch.matmul(dO, _T(t["Wo"])), H)
    dK3, dQ3, dZ = _decode_grad(K, Q, Z, Y, dY)
    dQ2, dK2, dV = _encode_grad(Q, K, V, Z, L2, dZ)
    ds, dKt, dVt = _encode_grad(t["seeds"][None], Kt, Vt, Q, L1, dQ3 + dQ2)
    Xt = X.reshape(B * N, C).t().contiguous()
    g = {"dX": torch.zeros_like(X), "dseeds": ds.sum(0),
         "dWo": torch.matmul(_merge(Y).reshape(B * N, C).t().contiguous(), dO.reshape(B * N, C))}
    for k, G in (("Wk", dK3 + dK2), ("Wv", dV), ("Wkt", dKt), ("Wvt", dVt)):
        G = _merge(G)
        g["dX"] += torch.matmul(G, _T(t[k]))
        g["d" + k] = torch.matmul(Xt, G.reshape(B * N, C))
    return g


def exact(case, seed):
    op, H = case["op"], case["H"]
    t = {k: v.double() for k, v in _inputs(case, seed).items()}
    X = t["X"]
    if op == "primitives":
        K, V = _heads(torch.matmul(X, t["Wk"]), H), _heads(torch.matmul(X, t["Wv"]), H)
        Z, lse = _encode(t["q"], K, V)
        return K, V, Z, lse, _merge(_decode(K, t["q"], Z))
    if op == "flare":
        K, V = _heads(torch.matmul(X, t["Wk"]), H), _heads(torch.matmul(X, t["Wv"]), H)
        Z, _ = _encode(t["seeds"][None], K, V)
        return torch.matmul(_merge(_decode(K, t["seeds"][None], Z)), t["Wo"])
    if op != "block":
        O, kept = _mixer(X, t, H)
        if op == "forward":
            return O
        g = _mixer_grad(X, t, H, kept, t["dO"])
        return g if op == "backward" else (O, g)
    mean = X.mean(-1, keepdim=True)
    r = 1 / (X.var(-1, unbiased=False, keepdim=True) + EPS).sqrt()
    xhat = (X - mean) * r
    Xn = xhat * t["gamma"] + t["beta"]
    O, kept = _mixer(Xn, t, H)
    g = _mixer_grad(Xn, t, H, kept, t["dO"])
    dXn = g["dX"]
    u = dXn * t["gamma"]
    g["dX"] = t["dO"] + r * (u - u.mean(-1, keepdim=True) - xhat * (u * xhat).mean(-1, keepdim=True))
    g["dgamma"], g["dbeta"] = (dXn * xhat).sum((0, 1)), dXn.sum((0, 1))
    return X + O, g
