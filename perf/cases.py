"""Performance cases of the GaLore path: what a training program has the library do.

A program keeps the weights W, the moments M and V, the projector P and a
workspace, and calls the library once per optimizer step and shape group: on one
weight matrix (a per-layer hook) or on a batch of same-shape matrices. The cases
stand for

* ``switch``  one ``galore_step`` at an update step (tau a multiple of T): the
              randomized subspace update, the sign match to the previous
              projector (optionally with the first moment re-expressed), then
              projection, Adam and the weight update;
* ``step``    one ``galore_step`` between updates, on the fixed projector;
* ``lowbit``  the step on a low-bit projector with 8-bit moments, through its
              three entry points;
* ``svd``     the exact SVD projector and its sign match.

Shapes, ranks and storage types are those of the Llama-shaped workloads of
60M to 7B parameters (hidden x hidden and hidden x intermediate, either way
round, r = hidden / 8 to hidden / 4, fp32 gradients for the small models, bf16
for the large ones), one matrix or a group of them.

Gradients: U diag(s) V^T + noise, U and V with orthonormal columns, s falling
geometrically by two decades over the kept rank and two more over as many
directions again, noise of 1e-6 per entry, rounded to the storage type. The
previous projector is the planted left (or right) vectors, so the columns of
the new one are determined up to rounding and keep their sign from one
implementation to another.
"""
import math

import numpy as np
import torch

import paper_2504_20437_amd as gl

T = 200                      # update interval
LR, ALPHA = 1e-3, 0.25
BETA1, BETA2, EPS = 0.9, 0.999, 1e-8
SKETCH_SEED = 20250430


def _case(name, kind, m, n, r, p, q, dtype, batch, aux=False, reexpress=False, bits=8):
    return {"name": name, "kind": kind, "m": m, "n": n, "r": r, "p": p, "q": q, "dtype": dtype, "batch": batch,
            "aux": aux, "reexpress": reexpress, "bits": bits}


def listed():
    return [
        # the smallest workload of the family: one matrix, launch and latency bound
        _case("switch-256x688-f32", "switch", 256, 688, 32, 8, 2, "f32", 1),
        # a 60M-shaped model stepped matrix by matrix from a per-parameter hook
        _case("step-512x1376-f32", "step", 512, 1376, 128, 8, 2, "f32", 1),
        # the 60M-shaped model's gate/up matrices as one group
        _case("switch-512x1376-f32-x16", "switch", 512, 1376, 128, 8, 2, "f32", 16),
        # 350M-shaped gate/up matrices, moments carried into the new basis
        _case("switch-1024x2736-f32-x6", "switch", 1024, 2736, 256, 16, 2, "f32", 6, reexpress=True),
        # 350M-shaped down matrices (right projector), every step but one in T
        _case("step-2736x1024-f32-x24", "step", 2736, 1024, 256, 16, 2, "f32", 24),
        # 1B-shaped gate/up matrices: rows of 5461 bf16 entries start on no 16-byte boundary
        _case("switch-2048x5461-bf16-x8", "switch", 2048, 5461, 512, 16, 2, "bf16", 8, aux=True),
        _case("step-2048x5461-bf16-x8", "step", 2048, 5461, 512, 16, 2, "bf16", 8),
        # one 7B-shaped gate/up matrix, from a per-layer hook
        _case("switch-4096x11008-bf16", "switch", 4096, 11008, 1024, 32, 2, "bf16", 1),
        # a group of them with the second stream: the throughput case
        _case("switch-4096x11008-bf16-x16", "switch", 4096, 11008, 1024, 32, 2, "bf16", 16, aux=True),
        # one 7B-shaped down matrix between updates (right projector)
        _case("step-11008x4096-bf16", "step", 11008, 4096, 1024, 32, 2, "bf16", 1),
        # 7B-shaped attention matrices with the int8 projector and 8-bit moments
        _case("lowbit-4096x4096-bf16-x8", "lowbit", 4096, 4096, 1024, 32, 2, "bf16", 8),
        # the exact SVD the randomized update replaces
        _case("svd-1024x1024-f32-x4", "svd", 1024, 1024, 256, 0, 0, "f32", 4),
    ]


def _update_flops(m, n, r, p, q):
    """products with the gradient, orthonormalisations and the small SVD"""
    s, l = min(m, n), max(m, n)
    k = min(r + p, s)
    return 2.0 * s * l * k * (2 + 2 * q) + 2.0 * k * k * ((q + 1) * s + q * l) + 8.0 * k ** 3 + 2.0 * s * k * r


def _flops(c):
    s, l, r, b = min(c["m"], c["n"]), max(c["m"], c["n"]), c["r"], c["batch"]
    f = 0.0
    if c["kind"] in ("switch", "step", "lowbit"):
        f += 4.0 * s * l * r
    if c["kind"] == "switch":
        f += _update_flops(c["m"], c["n"], r, c["p"], c["q"])
        if c["reexpress"]:
            f += 2.0 * s * r * r + 2.0 * r * r * l
    if c["kind"] == "svd":
        f += _update_flops(c["m"], c["n"], r, s - r, 0)
    return f * b


def draw(rng):
    largest = 1.3e13
    while True:
        kind = rng.choice(["switch", "switch", "switch", "step", "step", "step", "lowbit", "svd"])
        top = 1024 if kind == "svd" else 4096
        h = int(round(256 * (top / 256.0) ** rng.random()))
        if rng.random() < 0.6:
            h = max(256, h // 32 * 32)           # hidden sizes are mostly round ...
        f = h if rng.random() < 0.35 else int(round(h * rng.uniform(2.0, 3.5)))
        if rng.random() < 0.5:
            f = f // 16 * 16                     # ... intermediate sizes often not
        m, n = (h, f) if rng.random() < 0.6 else (f, h)
        s = min(m, n)
        r = max(16, int(s * rng.uniform(0.12, 0.26)))
        if rng.random() < 0.7:
            r = r // 16 * 16
        small = s < 1400
        dtype = rng.choice(["f32", "f32", "bf16"]) if small else rng.choice(["bf16", "bf16", "f32"])
        if kind == "lowbit":
            dtype = "bf16"
        c = _case("", kind, m, n, r, rng.choice([8, 16, 32]), rng.choice([1, 2, 2]), dtype, 1,
                  aux=rng.random() < 0.3, reexpress=rng.random() < 0.3, bits=rng.choice([8, 8, 4]))
        c["batch"] = int(round(32 ** rng.random()))
        if c["dtype"] == "f32" and c["batch"] * m * n > 2 ** 28:
            continue
        if kind == "svd" and c["batch"] > 8:
            continue
        if _flops(c) <= largest and c["batch"] * m * n <= 16 * 4096 * 11008:
            del c["name"]
            return c


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------


def _orthonormal(rows, cols, gen):
    z = torch.randn(rows, cols, generator=gen, device="cuda", dtype=torch.float64)
    for _ in range(2):
        c = torch.linalg.cholesky(z.T.contiguous() @ z)
        z = torch.linalg.solve_triangular(c, z.T.contiguous(), upper=False).T.contiguous()
    return z


def _gradients(c, gen):
    """(G, P_old): gradients of one planted pair, each under its own signed row
    and column permutation, and the planted vectors of the projected side."""
    m, n, r, b = c["m"], c["n"], c["r"], c["batch"]
    s = min(m, n)
    d = min(2 * r, s)
    U, V = _orthonormal(m, d, gen), _orthonormal(n, d, gen)
    sv = 10.0 ** (-2.0 * torch.arange(d, device="cuda", dtype=torch.float64) / r)
    base = ((U * sv) @ V.T.contiguous()).float()
    side = (U if m <= n else V)[:, :r].float()
    del U, V
    G = torch.empty((b, m, n), device="cuda", dtype=torch.float32 if c["dtype"] == "f32" else torch.bfloat16)
    P = torch.empty((b, s, r), device="cuda")
    for i in range(b):
        pr = torch.randperm(m, generator=gen, device="cuda")
        pc = torch.randperm(n, generator=gen, device="cuda")
        sr = torch.randint(0, 2, (m, 1), generator=gen, device="cuda").float() * 2 - 1
        sc = torch.randint(0, 2, (n, 1), generator=gen, device="cuda").float() * 2 - 1
        g = base.index_select(0, pr).index_select(1, pc) * sr * sc.T
        G[i] = g.add_(torch.randn(m, n, generator=gen, device="cuda"), alpha=1e-6)
        P[i] = side.index_select(0, pr) * sr if m <= n else side.index_select(0, pc) * sc
        # columns carry the sign the subspace update gives them
        top = P[i].abs().argmax(dim=0)
        P[i] *= torch.sign(P[i].gather(0, top[None]))
    return G, P


def _inputs(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    m, n, r, b = c["m"], c["n"], c["r"], c["batch"]
    l = max(m, n)
    x = {}
    x["G"], x["P"] = _gradients(c, gen)
    if c["kind"] == "svd":
        return x
    x["W"] = torch.randn((b, m, n), generator=gen, device="cuda") * 0.02
    # moments of a running state: the size of projected gradients of this scale
    scale = 1.0 / math.sqrt(l * r)
    x["M"] = torch.randn((b, r, l), generator=gen, device="cuda") * (0.5 * scale)
    x["V"] = (torch.randn((b, r, l), generator=gen, device="cuda") * scale) ** 2 + (0.1 * scale) ** 2
    return x


def _fp8_blocks(x, dtype, largest):
    """codes and power-of-two block scales of blocks of 2048 entries of each matrix"""
    b, r, l = x.shape
    nb = (r * l + 2047) // 2048
    flat = torch.zeros((b, nb * 2048), device="cuda")
    flat[:, :r * l] = x.reshape(b, -1)
    blocks = flat.view(b, nb, 2048)
    scale = torch.exp2(torch.ceil(torch.log2(blocks.abs().amax(dim=2).double() / largest))).float()
    codes = (blocks / scale[:, :, None]).to(dtype).view(torch.uint8).view(b, -1)[:, :r * l].reshape(b, r, l)
    return codes.contiguous(), scale.contiguous()


def prepare(case, seed):
    c = case
    m, n, r, b = c["m"], c["n"], c["r"], c["batch"]
    l = max(m, n)
    st = dict(c)
    st.update(_inputs(c, seed))
    dt = st["G"].dtype
    st["aux_stream"] = torch.cuda.Stream() if c["aux"] else None
    st["info"] = torch.zeros((b,), dtype=torch.int32, device="cuda")
    if c["kind"] in ("switch", "step"):
        st["flags"] = (gl.GALORE_STEP_ALIGN | (gl.GALORE_STEP_REEXPRESS if c["reexpress"] else 0)
                       if c["kind"] == "switch" else 0)
        need = gl.galore_step_workspace_size(m, n, r, c["p"], b, dt, st["flags"])
    elif c["kind"] == "lowbit":
        st["Pq"] = gl.galore_quantize_projector(st.pop("P"), c["bits"])
        st["state"] = gl.Adam8State(r, l, b)
        st["state"].M8, st["state"].Ms = _fp8_blocks(st.pop("M"), torch.float8_e4m3fn, 448.0)
        st["state"].V8, st["state"].Vs = _fp8_blocks(st.pop("V"), torch.float8_e5m2, 57344.0)
        st["R"] = torch.empty((b, r, l), device="cuda")
        need = max(gl.galore_project_quantized_workspace_size(m, n, r, b),
                   gl.galore_project_back_quantized_workspace_size(m, n, r, b))
    else:
        st["P_new"] = torch.empty_like(st["P"])
        st["sigma"] = torch.empty((b, r), device="cuda")
        need = gl.galore_svd_workspace_size(m, n, r, b, dt)
    st["workspace"] = torch.empty((max(need, 1),), dtype=torch.uint8, device="cuda")
    return st


def run(state):
    s = state
    if s["kind"] in ("switch", "step"):
        update = s["kind"] == "switch"
        gl.galore_step(s["G"], s["W"], s["P"], s["M"], s["V"], r=s["r"], p=s["p"], q=s["q"], seed=SKETCH_SEED,
                       tau=T if update else T + 1, T=T, beta1=BETA1, beta2=BETA2, eps=EPS, lr=LR, alpha=ALPHA,
                       flags=s["flags"], info=s["info"], workspace=s["workspace"], aux_stream=s["aux_stream"])
        if update:
            return s["W"], s["M"], s["V"], s["P"], s["info"]
        return s["W"], s["M"], s["V"]
    if s["kind"] == "lowbit":
        st = s["state"]
        R = gl.galore_project_quantized(s["Pq"], s["G"], R=s["R"], workspace=s["workspace"])
        N = gl.galore_lowrank_adam8_step(R, st, N=R, beta1=BETA1, beta2=BETA2, eps=EPS, t=T + 2)
        gl.galore_project_back_quantized(s["Pq"], N, s["W"], LR, ALPHA, workspace=s["workspace"])
        return s["W"], N, st.M8, st.Ms, st.V8, st.Vs
    P, sigma, info = gl.galore_svd_update(s["G"], s["r"], P=s["P_new"], sigma=s["sigma"], info=s["info"],
                                          workspace=s["workspace"], aux_stream=s["aux_stream"])
    gl.galore_align_projector(s["P"], P)
    return P, sigma, info


def work(case):
    c = case
    s, l, r, b = min(c["m"], c["n"]), max(c["m"], c["n"]), c["r"], c["batch"]
    g = s * l * (4 if c["dtype"] == "f32" else 2)
    if c["kind"] == "svd":
        by = g + 4 * s * r + 4 * s * r + 4 * r + 4      # G and P_old in, P, sigma and info out
    elif c["kind"] == "lowbit":
        # G, codes, scales, both moments in and out, W in and out, N out
        by = g + s * r * c["bits"] // 8 + 4 * r + 4 * r * l + 8 * s * l + 4 * r * l + 16 * (r * l // 2048 + 1)
    else:
        by = g + 8 * s * l + 16 * r * l + 4 * s * r     # G, W, M and V, P
        if c["kind"] == "switch":
            by += 4 * s * r
    return {"bytes": float(by) * b, "flops": _flops(c)}


def tolerance(case):
    # about four times what this path is from its 64-bit result: P 6e-5 (single
    # columns whose neighbours are close 1e-3, their largest entry 4e-3), the
    # exact SVD's P 1.5e-5 (2e-4), projected moments 6e-7 (6e-6); of the 8-bit
    # codes, those whose moment lies on a rounding boundary
    if case["kind"] == "switch":
        return {"rel": 5e-4, "max": 0.1}
    if case["kind"] == "svd":
        return {"rel": 1e-4, "max": 1e-2}
    if case["kind"] == "lowbit":
        return {"rel": 5e-6, "max": 1e-4, "differ": 2e-4}
    return {"rel": 5e-6, "max": 1e-4}


# --------------------------------------------------------------------------
# the same in 64 bits, from plain torch and numpy
# --------------------------------------------------------------------------


def _sketch(l, k, index):
    """Omega: Philox4x64-10 keyed by the seed, four rows of a column a block,
    Box-Muller pairs rounded to bf16"""
    nb = k * ((l + 3) // 4)
    # numpy steps its 256-bit counter before each block: start one before (0, index, 0, 0)
    start = (index << 64) - 1
    counter = [(start >> (64 * i)) & (2 ** 64 - 1) for i in range(4)]
    raw = np.random.Philox(counter=np.array(counter, dtype=np.uint64),
                           key=np.array([SKETCH_SEED, 0], dtype=np.uint64)).random_raw(4 * nb).reshape(nb, 2, 2)
    u1 = ((raw[:, :, 0] >> np.uint64(11)).astype(np.float64) + 1.0) * 2.0 ** -53
    u2 = (raw[:, :, 1] >> np.uint64(11)).astype(np.float64) * 2.0 ** -53
    rad = np.sqrt(-2.0 * np.log(u1))
    z = np.stack([rad * np.cos(2 * np.pi * u2), rad * np.sin(2 * np.pi * u2)], axis=2)
    om = torch.from_numpy(np.ascontiguousarray(z.reshape(k, -1)[:, :l].T)).cuda()
    return om.to(torch.bfloat16).double()


def _orth(y):
    for _ in range(2):
        c = torch.linalg.cholesky(y.T.contiguous() @ y)
        y = torch.linalg.solve_triangular(c, y.T.contiguous(), upper=False).T.contiguous()
    return y


def _top(Q, B, r):
    w, u = np.linalg.eigh((B @ B.T.contiguous()).cpu().numpy())
    u = torch.from_numpy(np.ascontiguousarray(u[:, ::-1][:, :r])).cuda()
    return (Q @ u if Q is not None else u), torch.from_numpy(np.sqrt(np.maximum(w[::-1][:r], 0.0)).copy()).cuda()


def _matched(P, P_old):
    ov = (P * P_old).sum(dim=0)
    return torch.where(ov < 0, -P, P)


def _f32(x):
    return float(np.float32(x))


def exact(case, seed):
    c = case
    m, n, r, b = c["m"], c["n"], c["r"], c["batch"]
    s, l = min(m, n), max(m, n)
    if b * m * n > 4 * 4096 * 11008 or (c["kind"] == "switch" and b * m * n > 2 * 4096 * 11008):
        return None
    x = _inputs(c, seed)
    A64 = (lambda i: x["G"][i].double()) if m <= n else (lambda i: x["G"][i].double().T.contiguous())
    outs = {k: [] for k in ("W", "M", "V", "P", "sigma", "N")}
    t = T + 1 if c["kind"] == "switch" else T + 2
    b1, b2, eps = _f32(BETA1), _f32(BETA2), _f32(EPS)
    for i in range(b):
        A = A64(i)
        P = x["P"][i].double()
        if c["kind"] == "svd":
            Pn, sg = _top(None, A, r)
            outs["P"].append(_matched(Pn, P))
            outs["sigma"].append(sg)
            continue
        M, V, W = x["M"][i].double(), x["V"][i].double(), x["W"][i].double()
        if c["kind"] == "switch":
            k = min(r + c["p"], s)
            Q = _orth(A @ _sketch(l, k, i))
            for _ in range(c["q"]):
                Z = _orth(A.T.contiguous() @ Q)
                Q = _orth(A @ Z)
            Pn, _ = _top(Q, Q.T.contiguous() @ A, r)
            Pn = _matched(Pn, P)
            if c["reexpress"]:
                M = (Pn.T.contiguous() @ P) @ M
            P = Pn
        elif c["kind"] == "lowbit":
            qmax = 127 if c["bits"] == 8 else 7
            sc = x["P"][i].abs().amax(dim=0) / float(qmax)
            P = (torch.round(x["P"][i] / sc).clamp(-qmax, qmax).double()) * sc.double()
            codes, scale = _fp8_blocks(x["M"][i:i + 1], torch.float8_e4m3fn, 448.0)
            M = (codes.view(torch.float8_e4m3fn).double().view(-1)
                 * scale.double().repeat_interleave(2048, dim=1).view(-1)[:r * l]).view(r, l)
            codes, scale = _fp8_blocks(x["V"][i:i + 1], torch.float8_e5m2, 57344.0)
            V = (codes.view(torch.float8_e5m2).double().view(-1)
                 * scale.double().repeat_interleave(2048, dim=1).view(-1)[:r * l]).view(r, l)
        R = P.T.contiguous() @ A
        M = b1 * M + (1 - b1) * R
        V = b2 * V + (1 - b2) * R * R
        N = (M / (1 - b1 ** t)) / (torch.sqrt(V / (1 - b2 ** t)) + eps)
        D = P @ N
        outs["W"].append(W - _f32(LR) * _f32(ALPHA) * (D if m <= n else D.T))
        outs["M"].append(M)
        outs["V"].append(V)
        outs["N"].append(N)
        outs["P"].append(P)
    o = {k: torch.stack(v) for k, v in outs.items() if v}
    if c["kind"] == "svd":
        return o["P"], o["sigma"], None
    if c["kind"] == "lowbit":
        return o["W"], o["N"], None, None, None, None
    if c["kind"] == "switch":
        return o["W"], o["M"], o["V"], o["P"], None
    return o["W"], o["M"], o["V"]
