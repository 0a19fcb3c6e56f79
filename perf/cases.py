"""The workloads this framework's speed is measured on.

Each case is what a user's program does with the library: whole iterations of
the 3D SDDMM / SpMM loop on one processor's block (pack, compute, reduce),
single products, graph-attention layers, and the localization of a new
pattern.  Inputs are seeded and made on the GPU: R-MAT (power-law), uniform
and banded patterns, U[-1, 1) values.

listed() gives the named cases, draw(rng) further ones of the same ranges;
prepare(case, seed) makes the inputs and the plan a program keeps, run(state)
is one pass through the public entry points, work(case) the bytes and
operations a pass cannot do without, exact(case, seed) the outputs of one pass
over the same inputs in 64-bit arithmetic, from plain torch alone.
"""
from __future__ import annotations

import math

import torch

from paper_2404_19638_amd import autograd as ag
from paper_2404_19638_amd import spc3d as spc

DEV = "cuda:0"


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # The smallest iteration: 4096 x 4096, 40,000 entries.  Latency and
        # launches count.
        dict(name="step tiny", op="step", pattern="uniform", n=4096, nnz=40_000, K=32, kz=32,
             k0=0, dtype="f32", form="fused"),
        # One processor's share of a power-law graph (2^24 vertices, degree 16,
        # 8 x 8 x 4 grid): the headline workload.
        dict(name="step share rmat", op="step", pattern="rmat", lg=24, deg=16, grid=8, K=128,
             kz=32, k0=32, dtype="f32", form="fused"),
        # The same block shape with flat degrees; the reduction at the owner is
        # folded into the pass, the faster form on such blocks.
        dict(name="step share uniform", op="step", pattern="uniform", n=1 << 21, nnz=4_012_517,
             K=128, kz=32, k0=32, dtype="f32", form="folded"),
        # A mesh-like block (two entries per row near the diagonal), bfloat16
        # operands, two slices along the third grid axis.
        dict(name="step banded bf16", op="step", pattern="banded", n=1 << 21, per_row=2,
             half=1 << 14, K=128, kz=64, k0=64, dtype="bf16", form="fused"),
        # K = 60 over Z = 2: rows of 30 values, not a multiple of 16 bytes;
        # SDDMM and SpMM called separately.
        dict(name="step ragged", op="step", pattern="rmat", lg=18, deg=16, grid=1, K=60, kz=30,
             k0=30, dtype="f32", form="separate"),
        # One of Z = 4 partial SDDMMs of K = 240, added into the running sum.
        dict(name="sddmm z-partial", op="sddmm", pattern="rmat", lg=19, deg=32, grid=1, kz=60,
             dtype="f32"),
        # The largest block: a whole graph of 2^22 vertices, K = 128, both
        # products of packed operands in one pass.
        dict(name="pass large", op="pass", pattern="rmat", lg=22, deg=32, grid=1, kz=128,
             dtype="f32"),
        # Inference of a graph-attention layer in bfloat16.
        dict(name="attention infer", op="infer", pattern="rmat", lg=18, deg=32, grid=1, kz=64,
             dtype="bf16"),
        # A training step's forward and backward of that layer, FP32, on a
        # large graph, and on a small one where launches count.
        dict(name="attention train", op="train", pattern="rmat", lg=20, deg=32, grid=1, kz=64,
             dtype="f32"),
        dict(name="attention train small", op="train", pattern="rmat", lg=11, deg=8, grid=1,
             kz=32, dtype="f32"),
        # Localization of a new pattern: the share block from COO, and a
        # medium graph from CSR with the column view that training needs.
        dict(name="setup share", op="setup", pattern="rmat", lg=24, deg=16, grid=8, source="coo",
             csc=False),
        dict(name="setup graph", op="setup", pattern="rmat", lg=16, deg=32, grid=1, source="csr",
             csc=True),
    ]


def _draw_pattern(rng, lg_most):
    kind = rng.choice(["rmat", "rmat", "uniform", "banded"])
    if kind == "rmat":
        lg = rng.randint(10, lg_most)
        return dict(pattern="rmat", lg=lg, deg=rng.randint(4, 32),
                    grid=1 if lg < 14 else rng.choice([1, 1, 2, 4]))
    n = int(round(2.0 ** rng.uniform(10, lg_most + 0.9)))
    if kind == "uniform":
        return dict(pattern="uniform", n=n, nnz=int(n * 2.0 ** rng.uniform(0, 5)))
    return dict(pattern="banded", n=n, per_row=rng.randint(2, 12),
                half=max(4, int(n * 2.0 ** rng.uniform(-10, -3))))


def draw(rng):
    op = rng.choice(["step", "step", "step", "sddmm", "pass", "infer", "train", "setup"])
    if op == "setup":
        c = dict(op=op, **_draw_pattern(rng, 19))
        c.update(source=rng.choice(["coo", "csr"]), csc=rng.random() < 0.5)
        return c
    if op in ("infer", "train"):
        c = dict(op=op, **_draw_pattern(rng, 18))
        c.update(kz=rng.choice([16, 32, 48, 60, 64, 96, 128]), dtype=rng.choice(["f32", "bf16"]))
        if c["dtype"] == "bf16" and c["kz"] == 60:
            c["kz"] = 64
        return c
    c = dict(op=op, **_draw_pattern(rng, 19))
    kz = rng.choice([15, 16, 24, 30, 32, 32, 40, 60, 64, 64, 80, 96, 120, 128])
    dtype = rng.choice(["f32", "f32", "bf16"])
    if op == "step":
        z = rng.choice([1, 2, 4])
        c.update(K=kz * z, kz=kz, k0=kz * rng.randrange(z), dtype=dtype,
                 form=rng.choice(["fused", "folded", "separate"]))
    else:
        c.update(kz=kz, dtype=dtype)
    return c


# ------------------------------------------------------------------- patterns

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _uniform(shape, g):
    return torch.empty(shape, dtype=torch.float32, device=DEV).uniform_(-1.0, 1.0, generator=g)


def _rmat_samples(lg, m, g):
    """m R-MAT samples on 2^lg vertices: (a, b, c, d) = (0.57, 0.19, 0.19,
    0.05) in 1/1024 steps, six levels from each 60-bit draw."""
    r = torch.zeros(m, dtype=torch.int32, device=DEV)
    c = torch.zeros(m, dtype=torch.int32, device=DEV)
    for l0 in range(0, lg, 6):
        bits = torch.randint(0, 1 << 60, (m,), generator=g, device=DEV)
        for _ in range(min(6, lg - l0)):
            t = (bits & 1023).to(torch.int32)
            bits >>= 10
            low = t >= 778                          # c or d: the row's bit
            right = low ^ (t >= 584) | (t >= 973)   # b or d: the column's bit
            r = (r << 1) | low
            c = (c << 1) | right
    return r, c


PATTERN_SEED = 2405


def _pattern(case, g):
    """(rows, cols, row_range, col_range): int64 global ids in caller order.
    Every seed gives a relabelling of one pattern of the case's kind, with its
    entries in another order (a COO file's order is any), so that a case has
    the same number of entries, rows and columns for every seed."""
    g0 = _gen(PATTERN_SEED)
    kind = case["pattern"]
    if kind == "rmat":
        lg, grid = case["lg"], case["grid"]
        n = 1 << lg
        span = n // grid
        bx, by = (5, 2) if grid == 8 else (grid - 1, 0)
        rlo, clo = bx * span, by * span
        perm = torch.randperm(n, generator=g0, device=DEV, dtype=torch.int64)
        left, keys = case["deg"] * n, []
        while left:
            m = min(left, 1 << 25)
            left -= m
            r, c = _rmat_samples(lg, m, g0)
            r, c = perm[r], perm[c]
            if grid > 1:
                keep = (r >= rlo) & (r < rlo + span) & (c >= clo) & (c < clo + span)
                r, c = r[keep], c[keep]
            keys.append((r - rlo) * span + (c - clo))
        keys = torch.unique(torch.cat(keys))
    else:
        n = span = case["n"]
        rlo = clo = 0
        if kind == "uniform":
            nnz = min(case["nnz"], n * n // 2)
            keys = torch.randint(0, n * n, (nnz + nnz // 2 + 64,), generator=g0, device=DEV)
            keys = torch.unique(keys)
            keys = keys[torch.randperm(keys.numel(), generator=g0, device=DEV)[:nnz]]
        else:
            r = torch.arange(n, device=DEV).repeat_interleave(case["per_row"])
            off = torch.randint(-case["half"], case["half"] + 1, (r.numel(),), generator=g0,
                                device=DEV)
            keys = torch.unique(r * n + (r + off).clamp_(0, n - 1))
    keys = keys[torch.randperm(keys.numel(), generator=g, device=DEV)]
    r, c = keys // span, keys % span
    if kind == "banded":   # a band stays one under a rotation
        turn = torch.randint(0, n, (1,), generator=g, device=DEV)
        r, c = (r + turn) % n, (c + turn) % n
    else:
        r = torch.randperm(span, generator=g, device=DEV)[r]
        c = torch.randperm(span, generator=g, device=DEV)[c]
    return r + rlo, c + clo, (rlo, rlo + span), (clo, clo + span)


# ----------------------------------------------------------------- the states

def _inputs(case, seed):
    """The inputs of a case: the pattern, its values and the dense operands,
    from the seed alone."""
    g = _gen(seed)
    rows, cols, rr, cr = _pattern(case, g)
    d = dict(rows=rows, cols=cols, rr=rr, cr=cr, vals=_uniform(rows.numel(), g))
    op = case["op"]
    if op == "step":
        d["A"] = _uniform((rr[1] - rr[0], case["K"]), g)
        d["B"] = _uniform((cr[1] - cr[0], case["K"]), g)
    elif op != "setup":
        R, C = torch.unique(rows).numel(), torch.unique(cols).numel()
        dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        if op in ("infer", "train"):
            # attention scores of order one
            s = math.sqrt(3.0) * case["kz"] ** -0.25
            d["Q"] = (_uniform((R, case["kz"]), g) * s).to(dt)
            d["Kf"] = (_uniform((C, case["kz"]), g) * s).to(dt)
            d["V"] = _uniform((C, case["kz"]), g).to(dt)
            if op == "train":
                d["dout"] = _uniform((R, case["kz"]), g)
        else:
            d["A"] = _uniform((R, case["kz"]), g).to(dt)
            d["B"] = _uniform((C, case["kz"]), g).to(dt)
            d["out"] = _uniform(rows.numel(), g)
    if op == "setup" and case["source"] == "csr":
        order = torch.argsort(rows, stable=True)
        d["rows"], d["cols"] = rows[order], cols[order].contiguous()
        counts = torch.bincount(d["rows"] - rr[0], minlength=rr[1] - rr[0])
        d["rowptr"] = torch.cat([counts.new_zeros(1), counts.cumsum(0)])
    return d


def prepare(case, seed):
    d = _inputs(case, seed)
    op = case["op"]
    s = dict(case=case)
    if op == "setup":
        s.update({k: d[k] for k in ("rows", "cols", "rr", "cr", "vals", "rowptr") if k in d})
        return s
    flags = spc.BUILD_CSC if op == "train" else 0
    plan = spc.plan_create_coo(d["rows"], d["cols"], d["rr"], d["cr"], flags)
    s["plan"] = plan
    if op in ("infer", "train"):
        for k in ("Q", "Kf", "V"):
            s[k] = d[k].requires_grad_(op == "train")
        if op == "train":
            s["dout"] = d["dout"]
        return s
    kz = case["kz"]
    s["vals"] = spc.permute_values(plan, spc.CALLER_TO_SLOT, d["vals"])
    if op == "step":
        dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
        s.update(A_src=d["A"], B_src=d["B"], dst=torch.zeros_like(d["A"]),
                 A=torch.empty((plan.R, kz), dtype=dt, device=DEV),
                 B=torch.empty((plan.C, kz), dtype=dt, device=DEV),
                 out=torch.empty(plan.nnz, device=DEV))
    else:
        s.update(A=d["A"], B=d["B"], out=d["out"])
    if op != "sddmm":
        s["Y"] = torch.empty((plan.R, kz), device=DEV)
        s["buf"] = torch.empty(spc.spmm_buffer_size(plan, 0, kz), dtype=torch.uint8, device=DEV)
    return s


# ------------------------------------------------------------------- one pass

def run(s):
    c = s["case"]
    op = c["op"]
    if op == "setup":
        flags = spc.BUILD_CSC if c["csc"] else 0
        if c["source"] == "csr":
            plan = spc.plan_create_csr(s["rowptr"], s["cols"], s["rr"], s["cr"], flags)
        else:
            plan = spc.plan_create_coo(s["rows"], s["cols"], s["rr"], s["cr"], flags)
        vals = spc.permute_values(plan, spc.CALLER_TO_SLOT, s["vals"])
        return dict(plan.maps(), vals=vals)
    plan = s["plan"]
    if op == "infer":
        with torch.no_grad():
            return dict(out=ag.gnn_attention(plan, s["Q"], s["Kf"], s["V"]))
    if op == "train":
        out = ag.gnn_attention(plan, s["Q"], s["Kf"], s["V"])
        dq, dk, dv = torch.autograd.grad(out, (s["Q"], s["Kf"], s["V"]), s["dout"])
        return dict(out=out.detach(), dQ=dq, dKf=dk, dV=dv)
    kz, A, B, vals, out = c["kz"], s["A"], s["B"], s["vals"], s["out"]
    if op == "sddmm":
        spc.sddmm(plan, vals, A, B, kz, out=out, mode=spc.ACCUMULATE)
        return dict(out=out)
    if op == "pass":
        spc.sddmm_spmm(plan, vals, A, B, kz, out=out, Y=s["Y"], buf=s["buf"])
        return dict(out=out, Y=s["Y"])
    k0, dst = c["k0"], s["dst"]
    spc.gather(plan, spc.ROWS, s["A_src"], k0, kz, out=A)
    spc.gather(plan, spc.COLS, s["B_src"], k0, kz, out=B)
    if c["form"] == "folded":
        spc.sddmm_spmm_scatter(plan, vals, A, B, dst, k0, kz, out=out, buf=s["buf"])
        return dict(out=out, dst=dst)
    if c["form"] == "fused":
        spc.sddmm_spmm(plan, vals, A, B, kz, out=out, Y=s["Y"], buf=s["buf"])
    else:
        spc.sddmm(plan, vals, A, B, kz, out=out)
        spc.spmm(plan, vals, B, 0, kz, out=s["Y"], buf=s["buf"])
    spc.scatter_reduce(plan, spc.ROWS, s["Y"], dst, k0)
    return dict(out=out, dst=dst)


# ----------------------------------------------------------- work and exact

def _sizes(case):
    """Expected (R, C, nnz) of a case's pattern: non-empty rows and columns
    and distinct entries."""
    kind = case["pattern"]
    if kind == "rmat":
        lg, grid = case["lg"], case["grid"]
        S = float(case["deg"]) * (1 << lg)
        nnz = 0.0
        for i in range(lg + 1):
            for j in range(lg - i + 1):
                cells = math.comb(lg, i) * math.comb(lg - i, j) * 2.0 ** j
                p = 0.57 ** i * 0.19 ** j * 0.05 ** (lg - i - j)
                nnz += cells * -math.expm1(-S * p)
        used = sum(math.comb(lg, u) * -math.expm1(-S / grid * 0.76 ** (lg - u) * 0.24 ** u)
                   for u in range(lg + 1))
        return used / grid, used / grid, nnz / grid ** 2
    n = case["n"]
    if kind == "uniform":
        nnz = min(case["nnz"], n * n // 2)
        used = n * -math.expm1(-nnz / n)
        return used, used, nnz
    cells = 2 * case["half"] + 1
    nnz = n * cells * -math.expm1(case["per_row"] * math.log1p(-1.0 / cells))
    return n, n * -math.expm1(-nnz / n), nnz


def work(case):
    """Every call's inputs read once and its outputs written once (packed rows
    and structure included; a row the block does not use is not read), and the
    multiply-adds of the products."""
    R, C, nnz = _sizes(case)
    op = case["op"]
    if op == "setup":
        ids = 16 * nnz if case["source"] == "coo" else 8 * nnz
        rng = (1 << case["lg"]) // case["grid"] if case["pattern"] == "rmat" else case["n"]
        if case["source"] == "csr":
            ids += 8 * rng
        csr = 8 * (R + C) + 8 * rng + 4 * R + 8 * nnz + 12 * nnz / 64
        csc = 4 * C + 8 * nnz + 12 * nnz / 64 if case["csc"] else 0
        return dict(bytes=ids + csr + csc + 8 * nnz, flops=0)
    kz, b = case["kz"], 4 if case["dtype"] == "f32" else 2
    if op in ("infer", "train"):
        fwd = kz * b * (R + 2 * C) + 4 * kz * R + 4 * (R + nnz)
        if op == "infer":
            return dict(bytes=fwd, flops=4 * kz * nnz)
        # the operands and the output gradient again, three gradients, both
        # views of the structure
        bwd = kz * b * (R + 2 * C) + 4 * kz * R + kz * b * (R + 2 * C) + 4 * (R + C + 2 * nnz)
        return dict(bytes=fwd + bwd, flops=14 * kz * nnz)
    if op == "sddmm":
        return dict(bytes=4 * R + 16 * nnz + kz * b * (R + C), flops=2 * kz * nnz)
    one = 4 * R + 12 * nnz + kz * b * (R + C)
    if op == "pass":
        return dict(bytes=one + 4 * kz * R, flops=4 * kz * nnz)
    pack = (8 + (4 + b) * kz) * (R + C)
    if case["form"] == "folded":
        total = pack + one + 8 * R + 8 * kz * R
    elif case["form"] == "fused":
        total = pack + one + 4 * kz * R + 8 * R + 12 * kz * R
    else:
        total = (pack + one + 4 * R + 8 * nnz + kz * b * C + 4 * kz * R
                 + 8 * R + 12 * kz * R)
    return dict(bytes=total, flops=4 * kz * nnz)


CHUNK = 1 << 28   # products per chunk of the 64-bit sums


def _dots(r, c, A, B):
    out = torch.empty(r.numel(), dtype=torch.float64, device=DEV)
    step = max(1, CHUNK // A.shape[1])
    for i in range(0, r.numel(), step):
        out[i:i + step] = (A[r[i:i + step]].double() * B[c[i:i + step]].double()).sum(1)
    return out


def _row_sums(n, r, w, c, X):
    """sum over the entries of each row r (ascending) of w * X[c]."""
    out = torch.zeros((n, X.shape[1]), dtype=torch.float64, device=DEV)
    step = max(1, CHUNK // X.shape[1])
    for i in range(0, r.numel(), step):
        ids, count = torch.unique_consecutive(r[i:i + step], return_counts=True)
        part = w[i:i + step, None] * X[c[i:i + step]].double()
        out[ids] += torch.segment_reduce(part, "sum", lengths=count, axis=0, unsafe=True)
    return out


def exact(case, seed):
    d = _inputs(case, seed)
    gr, r = torch.unique(d["rows"], return_inverse=True)
    gc, c = torch.unique(d["cols"], return_inverse=True)
    R, C = gr.numel(), gc.numel()
    order = torch.argsort(r * C + c, stable=True)
    r, c, v = r[order], c[order], d["vals"][order].double()
    op = case["op"]
    if op == "setup":
        names = ["gmap_r", "gmap_c", "lmap_r", "lmap_c", "rowptr", "colidx", "perm"]
        names += ["colptr", "rowidx_t", "slot_t"] if case["csc"] else []
        return dict({k: None for k in names}, vals=v)
    if op in ("infer", "train"):
        Q, Kf, V = d["Q"], d["Kf"], d["V"]
        e = _dots(r, c, Q, Kf)
        count = torch.bincount(r, minlength=R)
        m = torch.segment_reduce(e, "max", lengths=count, unsafe=True)
        a = torch.exp(e - m[r])
        a = a / torch.segment_reduce(a, "sum", lengths=count, unsafe=True)[r]
        out = _row_sums(R, r, a, c, V)
        if op == "infer":
            return dict(out=out)
        do = d["dout"].to(V.dtype)   # the gradient enters in the operands' type
        da = _dots(r, c, do, V)
        de = a * (da - torch.segment_reduce(a * da, "sum", lengths=count, unsafe=True)[r])
        t = torch.argsort(c, stable=True)
        return dict(out=out, dQ=_row_sums(R, r, de, c, Kf),
                    dKf=_row_sums(C, c[t], de[t], r[t], Q),
                    dV=_row_sums(C, c[t], a[t], r[t], do))
    if op == "step":
        ks = slice(case["k0"], case["k0"] + case["kz"])
        A = d["A"][gr - d["rr"][0], ks]
        B = d["B"][gc - d["cr"][0], ks]
        if case["dtype"] == "bf16":
            A, B = A.bfloat16(), B.bfloat16()
    else:
        A, B = d["A"], d["B"]
    out = v * _dots(r, c, A, B)
    if op == "sddmm":
        return dict(out=d["out"].double() + out)
    Y = _row_sums(R, r, v, c, B)
    if op == "pass":
        return dict(out=out, Y=Y)
    dst = torch.zeros(d["A"].shape, dtype=torch.float64, device=DEV)
    dst[gr - d["rr"][0], ks] = Y
    return dict(out=out, dst=dst)
