"""Performance cases of the per-rank SpMM path, through its public entry points.

Each case names one kind of call, the sparse matrix it works on and the dense
width and type.  Matrices are random draws of the families the framework is
used with: R-MAT graphs (power-law degrees, hubs at low ids; one block, or one
row panel of a distributed matrix), their symmetrised and degree-normalised
form (a graph-convolution layer) and uniform Erdos-Renyi panels.  Sizes follow
the repository's workloads: the 4096-vertex graph, a 131072-row panel of a
2^24-vertex matrix split over 128 ranks, the 2^21-vertex normalised graph.
Every plan runs with the tuning it has by default, as in the README's example.

Kinds of calls:
  forward  pack_B, spmm                               (inference, one product)
  train    shiro_spmm and its backward through autograd (a layer in training)
  step     pack_B, spmm, spmm_backward into packed gradient rows (a rank's step:
           the packed rows are what it sends back to their owners)
  replay   the step captured once and replayed as a HIP graph (serving loops)
  dvals    spmm_backward for the value gradients alone (learned edge weights)
  joint    JointSpMM.forward: the joint row/column strategy on one panel
  plan     partition, select_rows, prepare and the selection (a new pattern)
"""
from __future__ import annotations

import math

import torch

import paper_2512_20178_amd as shiro

_ABCD = (0.57, 0.19, 0.19, 0.05)  # R-MAT quadrant probabilities
_DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}


def _case(name, kind, graph, scale, degree, N, dtype, P=1, p=0):
    """graph: rmat | norm | er.  2^scale vertices, `degree` edge samples per row
    of the panel, panel p of P (P a power of two)."""
    c = {"kind": kind, "graph": graph, "scale": scale, "degree": degree, "N": N, "dtype": dtype, "P": P, "p": p}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # one layer of a small graph in training: every launch and host call counts
        _case("tiny_train_f32", "train", "rmat", 10, 8, 64, "f32", 4, 1),
        # the 4096-vertex single-block product, narrow features
        _case("small_forward_f32", "forward", "rmat", 12, 16, 32, "f32"),
        # the same graph's whole step as a captured graph
        _case("small_replay_f32", "replay", "rmat", 12, 16, 32, "f32"),
        # a new pattern: what a rank pays before its first training step
        _case("plan_panel", "plan", "rmat", 24, 32, 128, "f32", 128, 0),
        # one rank's training step on a power-law panel, the headline size
        _case("panel_step_f32", "step", "rmat", 24, 32, 128, "f32", 128, 0),
        # the same panel's product with bfloat16 features
        _case("panel_forward_bf16", "forward", "rmat", 24, 32, 128, "bf16", 128, 0),
        # a panel without hubs: almost every gathered row is used once
        _case("er_forward_f32", "forward", "er", 24, 32, 64, "f32", 128, 0),
        # a graph-convolution layer in training, the largest case
        _case("gcn_train_f32", "train", "norm", 21, 25, 128, "f32"),
        # wide features in bfloat16, training on a mid-size graph
        _case("wide_train_bf16", "train", "rmat", 20, 32, 256, "bf16"),
        # an output layer: as many columns as classes, not a multiple of anything
        _case("odd_train_f32", "train", "rmat", 18, 16, 47, "f32"),
        # gradients of edge weights alone
        _case("edge_grad_f32", "dvals", "rmat", 19, 32, 64, "f32"),
        # the joint row/column strategy on one rank's panel
        _case("joint_forward_f32", "joint", "rmat", 22, 32, 128, "f32", 32, 0),
    ]


def draw(rng):
    """One more case of the listed ranges: graphs of 2^10 to 2^21 vertices (or
    panels of up to 131072 rows of matrices of up to 2^24), widths of 16 to
    256 with a third of them odd or ragged, both types."""
    kind = rng.choice(["forward", "forward", "train", "train", "train", "step", "step", "replay", "dvals", "joint",
                       "plan"])
    if rng.random() < 0.35:
        N = int(round(math.exp(rng.uniform(math.log(16), math.log(256)))))
    else:
        N = rng.choice([16, 32, 48, 64, 96, 128, 192, 256])
    dtype = rng.choice(["f32", "f32", "bf16"])
    if kind == "joint" or (kind in ("forward", "step", "dvals", "plan") and rng.random() < 0.5):
        # one panel of a row-partitioned matrix
        graph = "rmat" if kind == "joint" else rng.choice(["rmat", "rmat", "er"])
        bits = rng.randint(12, 16 if kind == "joint" else 17)  # log2 of the panel's rows
        P = 1 << rng.randint(2, min(7, 24 - bits))
        return _case(None, kind, graph, bits + int(math.log2(P)), rng.randint(8, 40), N, dtype, P, 0)
    scale = rng.randint(10, 20)
    graph = rng.choice(["rmat", "rmat", "norm", "er"])
    degree = rng.randint(6, 32) if graph != "norm" else rng.randint(4, 16)
    if kind == "replay":
        scale = min(scale, 15)
    return _case(None, kind, graph, scale, degree, N, dtype, 1, 0)


# --------------------------------------------------------------------------
# matrices
# --------------------------------------------------------------------------
def _generator(seed, device):
    g = torch.Generator(device=device)
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _edges(case, g, device):
    """Edge samples of the case's panel: (global rows, global columns)."""
    L, Pb = case["scale"], int(math.log2(case["P"]))
    n = 1 << L
    rows = n >> Pb
    m = rows * case["degree"]
    if case["graph"] == "er":
        r = torch.randint(rows, (m,), generator=g, device=device) + case["p"] * rows
        return r, torch.randint(n, (m,), generator=g, device=device)
    a, b, c, d = _ABCD
    r = torch.zeros(m, dtype=torch.int64, device=device)
    col = torch.zeros(m, dtype=torch.int64, device=device)
    for level in range(L):
        u = torch.rand(m, generator=g, device=device)
        if level < Pb:  # the panel fixes the top row bits
            bit = (case["p"] >> (Pb - 1 - level)) & 1
            rb = torch.full_like(r, bit)
            cb = u >= (a / (a + b) if bit == 0 else c / (c + d))
        else:
            rb = (u >= a + b).long()
            cb = ((u >= a) & (u < a + b)) | (u >= a + b + c)
        r = (r << 1) | rb
        col = (col << 1) | cb.long()
    return r, col


def _matrix(case, seed, device):
    """CSR of the whole matrix with only the panel's rows filled: row_ptr
    int64, col int32 ascending in each row, vals float32.

    The edge samples are the case's own; the seed renames the vertices (an
    exclusive or on the low bits of the ids), so every seed has another matrix
    with the same numbers of nonzeros and of distinct columns."""
    n = 1 << case["scale"]
    r, c = _edges(case, _generator(0, device), device)
    if case["graph"] == "norm":
        r, c = torch.cat([r, c]), torch.cat([c, r])
    mix = (int(seed) * 2654435761 + 40503) % (1 << min(12, case["scale"] - int(math.log2(case["P"]))))
    key = torch.unique((r ^ mix) * n + (c ^ mix))
    r = torch.div(key, n, rounding_mode="floor")
    c = key - r * n
    counts = torch.bincount(r, minlength=n)
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=device)
    row_ptr[1:] = torch.cumsum(counts, 0)
    g = _generator(seed, device)
    if case["graph"] == "norm":
        deg = counts.double()
        vals = (1.0 / torch.sqrt(deg[r] * deg[c])).float()
    else:
        vals = torch.rand(key.numel(), generator=g, device=device)
    return row_ptr, c.int(), vals, g


def _inputs(case, seed, device):
    n, N = 1 << case["scale"], case["N"]
    rows = n // case["P"]
    row_ptr, col, vals, g = _matrix(case, seed, device)
    dt = _DTYPE[case["dtype"]]
    B = G = None
    if case["kind"] != "plan":
        B = torch.randn(n, N, generator=g, device=device).to(dt)
    if case["kind"] in ("train", "step", "replay", "dvals"):
        G = torch.randn(rows, N, generator=g, device=device).to(dt)
    return row_ptr, col, vals, B, G


# --------------------------------------------------------------------------
# the calls
# --------------------------------------------------------------------------
def _partition(s):
    c = s["case"]
    n = 1 << c["scale"]
    return shiro.partition(s["row_ptr"], s["col"], n, n, c["P"], c["p"])


def _step(s):
    plan = s["plan"]
    shiro.pack_B(plan, s["B"], out=s["Bp"])
    shiro.spmm(plan, s["vals"], s["Bp"], out=s["Y"])
    shiro.spmm_backward(plan, s["vals"], s["G"], s["Bp"], dBpacked=s["dBp"], dvals=s["dvals"])


def prepare(case, seed):
    dev = torch.device("cuda")
    row_ptr, col, vals, B, G = _inputs(case, seed, dev)
    s = {"case": dict(case), "row_ptr": row_ptr, "col": col, "vals": vals, "B": B, "G": G}
    kind, N, dt = case["kind"], case["N"], _DTYPE[case["dtype"]]
    n = 1 << case["scale"]
    if kind == "joint":
        js = shiro.JointSpMM(row_ptr, col, n, n, case["P"], case["p"])
        js.prepare(N, dt)
        s["js"] = js
    elif kind != "plan":
        plan = _partition(s)
        U, _ = shiro.select_rows(plan)
        shiro.prepare(plan, N, dt, ops=("spmm",) if kind == "forward" else ("spmm", "backward"))
        s["plan"] = plan
        if kind in ("step", "replay"):
            s["Bp"] = torch.empty(U, N, dtype=dt, device=dev)
            s["Y"] = torch.empty(n // case["P"], N, dtype=dt, device=dev)
            s["dBp"] = torch.empty(U, N, dtype=dt, device=dev)
            s["dvals"] = torch.zeros_like(vals)
        if kind == "dvals":
            s["Bp"] = shiro.pack_B(plan, B)
            s["dvals"] = torch.zeros_like(vals)
        if kind == "train":
            s["vals"] = vals.requires_grad_(True)
            s["B"] = B.requires_grad_(True)
        if kind == "replay":
            stream = torch.cuda.Stream()
            stream.wait_stream(torch.cuda.current_stream())
            with plan.capture(stream) as ids:
                _step(s)
            torch.cuda.current_stream().wait_stream(stream)
            s["graph"], s["stream"] = ids[0], stream
    torch.cuda.synchronize()
    return s


def run(state):
    s = state
    kind = s["case"]["kind"]
    if kind == "forward":
        Bp = shiro.pack_B(s["plan"], s["B"])
        return shiro.spmm(s["plan"], s["vals"], Bp)
    if kind == "train":
        Y = shiro.shiro_spmm(s["plan"], s["vals"], s["B"])
        dvals, dB = torch.autograd.grad(Y, (s["vals"], s["B"]), s["G"])
        return [Y.detach(), dvals, dB]
    if kind == "step":
        _step(s)
        return [s["Y"], s["dBp"], s["dvals"]]
    if kind == "replay":
        s["plan"].replay(s["graph"])
        return [s["Y"], s["dBp"], s["dvals"]]
    if kind == "dvals":
        shiro.spmm_backward(s["plan"], None, s["G"], s["Bp"], dvals=s["dvals"])
        return s["dvals"]
    if kind == "joint":
        return s["js"].forward(s["vals"], s["B"])
    plan = _partition(s)
    shiro.select_rows(plan)
    shiro.prepare(plan, s["case"]["N"], _DTYPE[s["case"]["dtype"]], ops=("spmm", "backward"))
    out = shiro.selection(plan)
    plan.close()
    return list(out)


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def _multinomial(L, k):
    out, left = 1, L
    for x in k:
        out *= math.comb(left, x)
        left -= x
    return out


def _hit(p, m):
    """Probability that an outcome of probability p occurs in m draws."""
    return -math.expm1(m * math.log1p(-p)) if p < 1 else 1.0


def _expected(case):
    """Expected (nonzeros, distinct columns) of the panel after duplicates
    are merged."""
    L, Pb = case["scale"], int(math.log2(case["P"]))
    n = 1 << L
    rows = n >> Pb
    m = rows * case["degree"]
    if case["graph"] == "er":
        nnz = rows * n * _hit(1.0 / (rows * n), m)
        return nnz, n * _hit(1.0 / n, nnz)
    a, b, c, d = _ABCD
    # the top Pb levels choose the column bit only
    ones = bin(case["p"]).count("1")
    zeros = Pb - ones
    q0, q1 = b / (a + b), d / (c + d)
    free = L - Pb
    nnz = 0.0
    sym = case["graph"] == "norm"
    for h0 in range(zeros + 1):
        for h1 in range(ones + 1):
            top = (q0 ** h0) * ((1 - q0) ** (zeros - h0)) * (q1 ** h1) * ((1 - q1) ** (ones - h1))
            ways = math.comb(zeros, h0) * math.comb(ones, h1)
            for i in range(free + 1):
                for j in range(free + 1 - i):
                    for k in range(free + 1 - i - j):
                        low = a ** i * b ** j * c ** k * d ** (free - i - j - k)
                        pr = top * low
                        if sym:  # (r, c) and (c, r) are both stored; b == c
                            pr *= 2 if j + k else 1
                        nnz += ways * _multinomial(free, (i, j, k)) * _hit(min(pr, 1.0), m)
    U = 0.0
    for h0 in range(zeros + 1):
        for h1 in range(ones + 1):
            top = (q0 ** h0) * ((1 - q0) ** (zeros - h0)) * (q1 ** h1) * ((1 - q1) ** (ones - h1))
            ways = math.comb(zeros, h0) * math.comb(ones, h1)
            for j in range(free + 1):
                pr = top * (b + d) ** j * (a + c) ** (free - j)
                U += ways * math.comb(free, j) * _hit(min(pr, 1.0), 2 * m if sym else m)
    return nnz, U


def work(case):
    nnz, U = _expected(case)
    N, n = case["N"], 1 << case["scale"]
    rows = n // case["P"]
    sz = 4 if case["dtype"] == "f32" else 2
    B, Y, dB = U * N * sz, rows * N * sz, n * N * sz
    pattern, vals = nnz * 4 + rows * 8, nnz * 4
    kind = case["kind"]
    if kind == "plan":  # the columns and row pointers in, the selection out
        return {"bytes": nnz * 4 + rows * 8 + U * 4 + nnz * 4 + case["P"] * 8, "flops": 0}
    if kind in ("forward", "joint"):
        return {"bytes": B + pattern + vals + Y, "flops": 2 * nnz * N}
    if kind == "dvals":
        return {"bytes": B + pattern + Y + vals, "flops": 2 * nnz * N}
    if kind == "train":  # B, dY, pattern and values in; Y, dB, dvals out
        return {"bytes": B + pattern + 2 * vals + 2 * Y + dB, "flops": 6 * nnz * N}
    # step, replay: B, dY, pattern, values in; Bpacked, Y, dBpacked, dvals out
    return {"bytes": 3 * B + pattern + 2 * vals + 2 * Y, "flops": 6 * nnz * N}


# --------------------------------------------------------------------------
# the same outputs in 64 bits
# --------------------------------------------------------------------------
def exact(case, seed):
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    row_ptr, col, vals, B, G = _inputs(case, seed, dev)
    n, N, P, p, kind = 1 << case["scale"], case["N"], case["P"], case["p"], case["kind"]
    rows, r0 = n // P, case["p"] * (n // P)
    row = torch.repeat_interleave(torch.arange(rows, device=dev), (row_ptr[1:] - row_ptr[:-1])[r0:r0 + rows])
    cols = col.long()
    uc, colmap = torch.unique(cols, return_inverse=True)
    if kind == "plan":
        K = n // P
        bounds = torch.arange(P + 1, device=dev) * K
        return [uc.int(), torch.searchsorted(uc, bounds).long(), colmap.int()]
    nnz = cols.numel()
    part = max(1, (1 << 28) // (8 * N))  # nonzeros at a time: 256 MB of products
    v64 = vals.double()
    Y = torch.zeros(rows, N, dtype=torch.float64, device=dev)
    packed = kind in ("step", "replay")
    dB = torch.zeros(uc.numel() if packed else n, N, dtype=torch.float64, device=dev)
    dvals = torch.zeros(nnz, dtype=torch.float64, device=dev)
    for k0 in range(0, nnz, part):
        k = slice(k0, min(nnz, k0 + part))
        if kind != "dvals":
            Y.index_add_(0, row[k], B[cols[k]].double() * v64[k, None])
        if G is not None:
            g = G[row[k]].double()
            dvals[k] = (g * B[cols[k]].double()).sum(1)
            if kind != "dvals":
                dB.index_add_(0, colmap[k] if packed else cols[k], g * v64[k, None])
    if kind in ("forward", "joint"):
        return Y
    if kind == "dvals":
        return dvals
    if kind == "train":
        return [Y, dvals, dB]
    return [Y, dB, dvals]
