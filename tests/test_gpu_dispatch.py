"""Which kernel a call takes, at the edges of the rules that choose it: widths
and strides beyond the nonzero walk, gathered matrices beyond 32-bit offsets,
outputs in place of inputs, infinities and NaN beside ragged tiles, gradients
written into uninitialised memory."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

# componentwise against |A||B|: float32 sums of up to a few thousand terms;
# bfloat16 operands and results rounded once each (2^-8 relative a rounding)
TOL = {torch.float32: 1e-5, torch.bfloat16: 1e-2}


@pytest.fixture(scope="module")
def shiro():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_20178_amd as s

    s._lib.load()
    return s


def _pattern(rows, cols, seed, density=0.2):
    rng = np.random.default_rng(seed)
    mask = rng.random((rows, cols)) < density
    mask[rows // 2, :] = False
    mask[0, :2] = True
    vals = rng.uniform(0.1, 1, size=(rows, cols)).astype(np.float32) * mask
    return synth.from_dense_pattern(vals, P=1, p=0, name="dispatch")


def _plan(shiro, A):
    Ad = A.to(torch.device("cuda"))
    plan = shiro.partition(Ad.row_ptr, Ad.col, A.n_rows, A.n_cols, 1, 0)
    U, _ = shiro.select_rows(plan)
    return plan, U, Ad


def test_more_column_tiles_than_a_grid_holds(shiro):
    """8,388,484 columns: 65536 tiles of the walk, one more than a grid may
    have in y; products and gradients still run (wider tiles)."""
    N = 128 * 65535 + 4
    rp = torch.tensor([0, 2, 2, 3], device="cuda")
    col = torch.tensor([0, 2, 1], dtype=torch.int32, device="cuda")
    vals = torch.tensor([2.0, -1.0, 3.0], device="cuda")
    plan = shiro.partition(rp, col, 3, 3, 1, 0)
    shiro.select_rows(plan)
    B = torch.arange(N, dtype=torch.float32, device="cuda") % 251
    B = torch.stack([B, B + 1, B + 2])
    Bp = shiro.pack_B(plan, B)
    Y = shiro.spmm(plan, vals, Bp)
    assert torch.equal(Y, torch.stack([2 * B[0] - B[2], torch.zeros_like(B[0]), 3 * B[1]]))
    dBp = torch.empty_like(Bp)
    shiro.spmm_backward(plan, vals, Y, None, dBpacked=dBp)
    assert torch.equal(dBp, torch.stack([2 * Y[0], 3 * Y[2], -Y[0]]))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N", [1, 2, 3, 72, 136, 200, 260, 264, 513, 520, 1030])
def test_sampled_product_kernels(shiro, N, dtype):
    """dvals alone: by default (lane groups up to 64 columns, the walk where
    its tiles are full or rows are no whole 16-byte pieces, else the row
    kernel), and with either kernel asked for, whose knobs then count."""
    A = _pattern(150, 200, N)
    plan, U, Ad = _plan(shiro, A)
    Ac = oracle.Csr.from_synth(A)
    B = synth.dense(A.n_cols, N, N, synth.STREAM_B).to(dtype)
    G = synth.dense(A.n_rows, N, N, synth.STREAM_DY).to(dtype)
    Bn, Gn = B.float().numpy(), G.float().numpy()
    ref, den = oracle.sddmm(Ac, Gn, Bn, None), oracle.sddmm(Ac, Gn, Bn, None, abs_mode=True)
    default = shiro.get_tuning(plan, "sddmm", N, dtype)
    if N > 64:
        walk = N in (72, 513) if dtype == torch.float32 else N in (72, 136, 200, 260, 513)
        walk &= not (dtype == torch.float32 and N == 513)  # five tiles
        assert default["group_rows"] == int(walk)
    knobs = [default, dict(default, group_rows=1, lanes=16), dict(default, group_rows=1, lanes=32)]
    knobs += [dict(default, group_rows=0, lanes=lanes, unroll=u, wg_per_cu=w, chunk=c)
              for lanes, u, w, c in ((8, 1, 1, 16), (16, 4, 32, 100), (32, 1, 2, 4096), (64, 2, 8, 128), (64, 4, 16, 64))]
    for pad in (0, 1):
        Bp = shiro.pack_B(plan, B.cuda(), out=torch.empty(U, N + pad, dtype=dtype, device="cuda")[:, :N])
        Gd = torch.zeros(A.n_rows, N + pad, dtype=dtype, device="cuda")[:, :N].copy_(G)
        for t in knobs:
            shiro.set_tuning(plan, "sddmm", N, dtype, **t)
            dvals = torch.full((A.nnz,), float("nan"), device="cuda")
            shiro.spmm_backward(plan, None, Gd, Bp, dvals=dvals)
            assert oracle.rel_err(dvals.cpu().numpy(), ref, den) <= 1e-5, (pad, t)


def _reused(n=1 << 17, deg=20, part=2 / 3):
    """2.6M nonzeros, 20 a row, on the given part of the columns: rows gathered
    many times, unevenly where some columns are not used at all."""
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    step = n // deg
    col = torch.randint(int(step * part), (n, deg), generator=g, device="cuda") + torch.arange(deg, device="cuda") * step
    row_ptr = torch.arange(0, n * deg + 1, deg, device="cuda")
    vals = torch.rand(n * deg, generator=g, device="cuda") + 0.1
    return row_ptr, col, vals


def _check_step(shiro, plan, col, vals, N, dtype, seed=0, pad=0):
    """Forward, dBpacked and dvals of a pattern with the same number of
    nonzeros in every row against float64 sums."""
    n, deg = col.shape
    U = plan.info()["U"]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def dense(rows):
        out = torch.empty(rows * (N + pad) + pad, dtype=dtype, device="cuda")[pad:].view(rows, N + pad)[:, :N]
        return out.copy_(torch.rand(rows, N, generator=g, device="cuda") + 0.1)

    uc, _, cm = shiro.selection(plan)
    cm = cm.long()
    Bp, G = dense(U), dense(n)
    Y, dBp = dense(n).fill_(float("nan")), dense(U).fill_(float("nan"))
    dvals = torch.full_like(vals, float("nan"))
    shiro.spmm(plan, vals, Bp, out=Y)
    shiro.spmm_backward(plan, vals, G, Bp, dBpacked=dBp, dvals=dvals)
    alone = torch.full_like(vals, float("nan"))
    shiro.spmm_backward(plan, None, G, Bp, dvals=alone)
    # every term is positive, so a result's size is its sum of absolute terms
    rows = torch.arange(n, device="cuda").repeat_interleave(deg)
    want = torch.zeros(n, N, dtype=torch.float64, device="cuda")
    dwant = torch.zeros(U, N, dtype=torch.float64, device="cuda")
    part = max(1, (1 << 26) // N)
    for k0 in range(0, vals.numel(), part):
        k = slice(k0, k0 + part)
        v, b, y = vals[k, None].double(), Bp[cm[k]].double(), G[rows[k]].double()
        want.index_add_(0, rows[k], v * b)
        dwant.index_add_(0, cm[k], v * y)
        dv = (b * y).sum(1)
        for got in (dvals[k], alone[k]):
            assert float(((got.double() - dv) / dv).abs().max()) <= TOL[torch.float32]
    assert float(((Y.double() - want) / want).abs().max()) <= TOL[dtype]
    assert float(((dBp.double() - dwant) / dwant).abs().max()) <= TOL[dtype]


@pytest.mark.parametrize("dtype,N,lanes", [(torch.float32, 72, 32), (torch.float32, 128, 16), (torch.float32, 320, 16),
                                           (torch.bfloat16, 136, 32), (torch.bfloat16, 256, 16)])
def test_tiles_of_reused_rows(shiro, dtype, N, lanes):
    """256-byte tiles where rows are reused unevenly, but not for rows that one
    512-byte tile holds, and never where they would take the value gradients out
    of the backward's walk (N = 320: five such tiles)."""
    row_ptr, col, vals = _reused(part=1)
    n = col.shape[0]
    plan = shiro.partition(row_ptr, col.reshape(-1).int(), n, n, 1, 0)
    shiro.select_rows(plan)
    assert shiro.get_tuning(plan, "spmm", N, dtype)["lanes"] == 32
    row_ptr, col, vals = _reused()
    n = col.shape[0]
    plan = shiro.partition(row_ptr, col.reshape(-1).int(), n, n, 1, 0)
    shiro.select_rows(plan)
    for k in ("spmm", "spmm_t"):
        assert shiro.get_tuning(plan, k, N, dtype)["lanes"] == lanes
    shiro.prepare(plan, N, dtype)
    _check_step(shiro, plan, col, vals, N, dtype)
    if N == 320:  # in the walk: the dots' error is that of sums over its tiles, and one launch less
        from torch.profiler import ProfilerActivity, profile

        Bp, G = torch.rand(plan.info()["U"], N, device="cuda"), torch.rand(n, N, device="cuda")
        dBp, dvals = torch.empty_like(Bp), torch.empty_like(vals)
        shiro.spmm_backward(plan, vals, G, Bp, dBpacked=dBp, dvals=dvals)
        torch.cuda.synchronize()
        with profile(activities=[ProfilerActivity.CUDA]) as prof:
            shiro.spmm_backward(plan, vals, G, Bp, dBpacked=dBp, dvals=dvals)
            torch.cuda.synchronize()
        assert not any("k_sddmm" in e.key for e in prof.key_averages())


def _few(n_rows=1 << 16, deg=20, n_cols=1 << 21):
    """1.3M nonzeros over 2M columns: a column holds 1.3 of them at most."""
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    step = n_cols // deg
    col = torch.randint(step, (n_rows, deg), generator=g, device="cuda") + torch.arange(deg, device="cuda") * step
    row_ptr = torch.arange(0, n_rows * deg + 1, deg, device="cuda")
    vals = torch.rand(n_rows * deg, generator=g, device="cuda") + 0.1
    return row_ptr, col, vals, n_cols


@pytest.mark.parametrize("dtype,N,forward,backward", [
    (torch.bfloat16, 1, 64, 64), (torch.bfloat16, 2, 0, 64), (torch.bfloat16, 7, 64, 64), (torch.bfloat16, 8, 0, 0),
    (torch.bfloat16, 9, 96, 96), (torch.bfloat16, 12, 0, 96), (torch.bfloat16, 15, 96, 96), (torch.bfloat16, 17, 0, 0),
    (torch.float32, 1, 0, 64), (torch.float32, 3, 0, 64), (torch.float32, 4, 0, 0), (torch.float32, 7, 0, 0)])
def test_narrow_rows(shiro, dtype, N, forward, backward):
    """Narrow products of patterns above 2^20 nonzeros: the windowed walk with
    chunks of its own (0: the nonzero walk), on rows that are reused and on
    rows that are not, whole rows and padded ones."""
    row_ptr, col, vals = _reused()
    n = col.shape[0]
    plan = shiro.partition(row_ptr, col.reshape(-1).int(), n, n, 1, 0)
    shiro.select_rows(plan)
    for k, chunk in (("spmm", forward), ("spmm_t", backward)):
        t = shiro.get_tuning(plan, k, N, dtype)
        assert t["group_rows"] == (3 if chunk else 2) and (not chunk or t["chunk"] == chunk)
    shiro.prepare(plan, N, dtype)
    for pad in (0, 1):
        _check_step(shiro, plan, col, vals, N, dtype, pad=pad)
    out = torch.empty(n, N, dtype=dtype, device="cuda")
    Bp = torch.rand(plan.info()["U"], N, device="cuda").to(dtype)
    assert torch.equal(shiro.spmm_noalloc(plan, vals, Bp, out), shiro.spmm(plan, vals, Bp))
    row_ptr, col, vals, n_cols = _few()
    plan = shiro.partition(row_ptr, col.reshape(-1).int(), col.shape[0], n_cols, 1, 0)
    shiro.select_rows(plan)
    t = shiro.get_tuning(plan, "spmm_t", N, dtype)
    short = bool(backward) or (dtype == torch.float32 and N < 12 and N % 4 != 0)
    assert t["group_rows"] == (3 if short else 2) and (not short or t["chunk"] == (256 if N < 8 else 128))
    _check_step(shiro, plan, col, vals, N, dtype)


@pytest.mark.parametrize("dtype,N,windowed", [
    (torch.float32, 128, False), (torch.float32, 132, True), (torch.float32, 160, True), (torch.float32, 192, False),
    (torch.float32, 200, True), (torch.float32, 201, False), (torch.float32, 252, True), (torch.float32, 256, False),
    (torch.bfloat16, 264, True), (torch.bfloat16, 260, False), (torch.bfloat16, 384, False)])
def test_partly_filled_tiles(shiro, dtype, N, windowed):
    """Rows of one to two tiles above 2^20 nonzeros: the windowed walk where
    the second tile is mostly idle or rows are no whole lines; operands at odd
    addresses run as well, eagerly and in a capture that was prepared for
    aligned ones."""
    row_ptr, col, vals, n_cols = _few(n_cols=1 << 19)
    plan = shiro.partition(row_ptr, col.reshape(-1).int(), col.shape[0], n_cols, 1, 0)
    shiro.select_rows(plan)
    for k in ("spmm", "spmm_t"):
        assert (shiro.get_tuning(plan, k, N, dtype)["group_rows"] == 3) == windowed
    shiro.prepare(plan, N, dtype)
    for pad in (0, 1):
        _check_step(shiro, plan, col, vals, N, dtype, pad=pad)
    fresh = shiro.partition(row_ptr, col.reshape(-1).int(), col.shape[0], n_cols, 1, 0)
    U, _ = shiro.select_rows(fresh)
    shiro.prepare(fresh, N, dtype)
    n = col.shape[0]
    store = [torch.rand(r * N + 1, device="cuda").to(dtype)[1:].view(r, N) for r in (U, n)]
    Bp, G = store
    Y, dBp, dvals = torch.empty_like(G), torch.empty_like(Bp), torch.zeros_like(vals)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        shiro.spmm(fresh, vals, Bp, out=Y)
        shiro.spmm_backward(fresh, vals, G, Bp, dBpacked=dBp, dvals=dvals)
    for _ in range(2):
        graph.replay()
        torch.cuda.synchronize()
        tol = TOL[dtype]
        assert float((Y.double() / shiro.spmm(plan, vals, Bp).double() - 1).abs().max()) <= 2 * tol
        want, dv = torch.empty_like(Bp), torch.zeros_like(vals)
        shiro.spmm_backward(plan, vals, G, Bp, dBpacked=want, dvals=dv)
        assert float((dBp.double() - want.double()).abs().max() / want.double().abs().max()) <= 2 * tol
        assert float(((dvals - dv) / dv).abs().max()) <= 1e-5


def test_tunings_of_earlier_kernels_are_not_applied(shiro, tmp_path, monkeypatch):
    """A tuning file keeps results across libraries.  Lines written for kernels
    that are gone (no generation in their key) are not applied; this library's
    own are."""
    A, N = synth.small_rmat(9, 8), 96
    plan, U, Ad = _plan(shiro, A)
    arch = torch.cuda.get_device_properties(0).gcnArchName.replace(" ", "_").replace(":", "_")
    cache = tmp_path / "tune.txt"
    old = [f"{arch}|rows={A.n_rows}|nnz={A.nnz}|U={U}|P=1|N={N}|dt=0|k={k} 4099 8 1 {g} 1 3" for k, g in ((0, 1), (1, 2), (2, 0))]
    cache.write_text("\n".join(old) + "\n")
    monkeypatch.setenv("SHIRO_TUNE_CACHE", str(cache))
    shiro.autotune(plan, N)
    got = {k: shiro.get_tuning(plan, k, N) for k in ("spmm", "spmm_t", "sddmm")}
    assert all(t["chunk"] != 4099 for t in got.values())
    lines = cache.read_text().splitlines()
    assert lines[:3] == old and len(lines) == 6
    keep = [ln.split(" ")[0] + " 4099 8 1 2 1 3 0" for ln in lines[3:5]]
    cache.write_text("\n".join(keep) + "\n")
    again, _, _ = _plan(shiro, A)
    shiro.autotune(again, N, ops=("spmm",))
    assert shiro.get_tuning(again, "spmm", N)["chunk"] == 4099


def _strided(rows, N, stride, seed, dtype=torch.float32):
    """rows x N with `stride` elements between rows, filled from seed."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    t = torch.empty((rows - 1) * stride + N, dtype=dtype, device="cuda").as_strided((rows, N), (stride, 1))
    t.copy_(torch.rand(rows, N, generator=g, device="cuda") + 0.1)
    return t


def _tight(t):
    return t.contiguous() if t.stride(0) == t.shape[1] else t.clone(memory_format=torch.contiguous_format)


@pytest.mark.parametrize("dtype,N,rows,stride", [
    (torch.float32, 96, 3, (1 << 30) + 4),     # rows 4 GB apart: the row kernel
    (torch.float32, 130, 3, (1 << 30) + 1),
    (torch.bfloat16, 160, 3, (1 << 31) + 8),
    (torch.float32, 96, 80, 1 << 24),          # 5 GB of rows: gathers of 64-bit offsets
    (torch.float32, 33, 80, (1 << 24) + 1),
    (torch.bfloat16, 160, 80, 1 << 25),
    (torch.bfloat16, 31, 80, (1 << 25) + 1),
])
def test_rows_far_apart(shiro, dtype, N, rows, stride):
    """Operands whose rows, or whole extent, lie beyond 32-bit byte offsets
    give what tight copies of them give."""
    A = _pattern(rows, rows, 5, density=0.5 if rows == 3 else 0.2)
    plan, U, Ad = _plan(shiro, A)
    tol = TOL[dtype]

    def close(a, b, t):
        a, b = a.double(), b.double()
        return float(((a - b).abs() / b.abs().clamp_min(1e-30)).max()) <= t

    Bp = _strided(U, N, stride, 1, dtype)
    Y = shiro.spmm(plan, Ad.vals, Bp)
    Bt = _tight(Bp)
    assert close(Y, shiro.spmm(plan, Ad.vals, Bt), 2 * tol)
    G = _strided(A.n_rows, N, stride, 2, dtype) if rows > 3 else (torch.rand(A.n_rows, N, device="cuda") + 0.1).to(dtype)
    Gt = _tight(G)
    want, dv = torch.empty_like(Bt), torch.zeros(A.nnz, device="cuda")
    shiro.spmm_backward(plan, Ad.vals, Gt, Bt, dBpacked=want, dvals=dv)
    got, gv = torch.empty_like(Bt), torch.zeros(A.nnz, device="cuda")
    shiro.spmm_backward(plan, Ad.vals, G, Bp, dBpacked=got, dvals=gv)
    assert close(got, want, 2 * tol) and close(gv, dv, 2e-5)
    gv.fill_(float("nan"))
    shiro.spmm_backward(plan, None, G, Bp, dvals=gv)
    assert close(gv, dv, 2e-5)
    del Bp, G
    out = _strided(A.n_rows, N, stride, 3, dtype) if rows == 3 else torch.empty_like(Gt)
    shiro.spmm(plan, Ad.vals, Bt, out=out)  # written rows far apart
    assert close(_tight(out), shiro.spmm(plan, Ad.vals, Bt), 2 * tol)


@pytest.mark.parametrize("N", [32, 64, 130, 200])
def test_gradients_in_place_of_values(shiro, N):
    """dvals may be the very array of the values (and so replace them): small
    patterns whose walk would read and write through the permutation, and wider
    ones."""
    A = synth.small_rmat(10, 16)
    plan, U, Ad = _plan(shiro, A)
    Bp = synth.dense(U, N, 1, synth.STREAM_B).cuda()
    G = synth.dense(A.n_rows, N, 2, synth.STREAM_DY).cuda()
    want, dv = torch.empty(U, N, device="cuda"), torch.zeros(A.nnz, device="cuda")
    shiro.spmm_backward(plan, Ad.vals, G, Bp, dBpacked=want, dvals=dv)
    got, both = torch.empty(U, N, device="cuda"), Ad.vals.clone()
    shiro.spmm_backward(plan, both, G, Bp, dBpacked=got, dvals=both)
    assert torch.equal(got, want)
    assert torch.equal(both, dv)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N", [5, 33, 47, 65, 129, 255])
def test_infinities_and_nan_stay_in_their_columns(shiro, N, dtype):
    """Not-a-numbers and infinities in some columns, the shared columns of a
    ragged tile's last lanes among them, reach exactly the results that their
    columns and rows contribute to."""
    A = _pattern(60, 70, N)
    plan, U, Ad = _plan(shiro, A)
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    Bp = (torch.rand(U, N, generator=g, device="cuda") + 0.1).to(dtype)
    G = (torch.rand(60, N, generator=g, device="cuda") + 0.1).to(dtype)
    uc, _, cm = shiro.selection(plan)
    rows = torch.repeat_interleave(torch.arange(60, device="cuda"), Ad.row_ptr[1:] - Ad.row_ptr[:-1])
    for col in sorted({0, N // 2, N - 4, N - 2, N - 1}):
        X, Z = Bp.clone(), G.clone()
        X[U // 2, col], Z[7, col] = float("nan"), float("inf")
        Y = shiro.spmm(plan, Ad.vals, X)
        hit = torch.zeros(60, dtype=torch.bool, device="cuda")
        hit[rows[cm.long() == U // 2]] = True
        bad = torch.isnan(Y)
        assert torch.equal(bad[:, col], hit) and int(bad.sum()) == int(hit.sum())
        dBp, dvals = torch.empty_like(X), torch.zeros(A.nnz, device="cuda")
        shiro.spmm_backward(plan, Ad.vals, Z, X, dBpacked=dBp, dvals=dvals)
        alone = torch.zeros(A.nnz, device="cuda")
        shiro.spmm_backward(plan, None, Z, X, dvals=alone)
        inf = torch.zeros(U, dtype=torch.bool, device="cuda")
        inf[cm.long()[rows == 7]] = True
        assert torch.equal(torch.isinf(dBp)[:, col], inf) and int((~torch.isfinite(dBp)).sum()) == int(inf.sum())
        nan, infd = cm.long() == U // 2, rows == 7
        for dv in (dvals, alone):
            assert torch.equal(torch.isnan(dv), nan)
            assert torch.equal(torch.isinf(dv), infd & ~nan)


@pytest.mark.parametrize("dtype,N", [(torch.float32, 16), (torch.float32, 200), (torch.bfloat16, 40), (torch.bfloat16, 300)])
def test_uninitialised_gradients_are_written_whole(shiro, dtype, N):
    """Where every column of the matrix occurs, autograd hands the backward an
    uninitialised dB, and where the plan holds every value an uninitialised
    dvals: no stale entry is left, for rows in one chunk and rows cut by many,
    one column tile and several."""
    rng = np.random.default_rng(N)
    n = 300
    mask = rng.random((n, n)) < 0.03
    mask[np.arange(n), np.arange(n)] = True  # every column occurs
    mask[:, 17] = rng.random(n) < 0.9        # cut by many chunks
    A = synth.from_dense_pattern((rng.uniform(0.1, 1, size=(n, n)) * mask).astype(np.float32), P=1, p=0, name="full")
    plan, U, Ad = _plan(shiro, A)
    assert U == n == plan.info()["n_cols"] and plan._whole
    for chunk in (None, 16):
        if chunk:
            shiro.set_tuning(plan, "spmm_t", N, dtype, chunk=chunk)
        B = synth.dense(n, N, 0, synth.STREAM_B).to(dtype).cuda()
        G = synth.dense(n, N, 0, synth.STREAM_DY).to(dtype).cuda()
        vals, Bl = Ad.vals.clone().requires_grad_(True), B.clone().requires_grad_(True)
        Y = shiro.shiro_spmm(plan, vals, Bl)
        stale = [torch.full((n * N,), float("nan"), dtype=dtype, device="cuda") for _ in range(4)]
        stale += [torch.full((A.nnz,), float("nan"), device="cuda") for _ in range(4)]
        del stale  # what the allocator hands out next
        dvals, dB = torch.autograd.grad(Y, (vals, Bl), G)
        Ac, Bn, Gn = oracle.Csr.from_synth(A), B.float().cpu().numpy(), G.float().cpu().numpy()
        assert oracle.rel_err(dB.float().cpu().numpy(), oracle.spmm_t(Ac, Gn, None),
                              oracle.spmm_t(Ac, Gn, None, abs_mode=True)) <= TOL[dtype]
        assert oracle.rel_err(dvals.cpu().numpy(), oracle.sddmm(Ac, Gn, Bn, None),
                              oracle.sddmm(Ac, Gn, Bn, None, abs_mode=True)) <= TOL[torch.float32]


def test_full_size_kernels_agree(shiro):
    """All 131072 rows, 1.2M packed columns and 4.15M values of the 2^24 R-MAT
    panel: the nonzero walk against the row kernel and the windowed walk, which
    sum in another order, componentwise against the sums of absolute terms."""
    A = synth.config2(device=torch.device("cuda"))
    N = 128
    plan = shiro.partition(A.row_ptr, A.col, A.n_rows, A.n_cols, A.P, A.p)
    U, _ = shiro.select_rows(plan)
    B = synth.dense(A.n_cols, N, 0, synth.STREAM_B, device="cuda")
    Bp = shiro.pack_B(plan, B)
    del B
    G = synth.dense(plan.info()["rows"], N, 0, synth.STREAM_DY, device="cuda")

    def run(vals, Bp, G, grp):
        for k in ("spmm", "spmm_t"):
            shiro.set_tuning(plan, k, N, group_rows=grp, chunk=256, lanes=32, unroll=4)
        Y, dBp, dv = shiro.spmm(plan, vals, Bp), torch.empty_like(Bp), torch.zeros_like(vals)
        shiro.spmm_backward(plan, vals, G, Bp, dBpacked=dBp, dvals=dv)
        return Y, dBp, dv

    den = run(A.vals.abs(), Bp.abs(), G.abs(), 0)
    walk = run(A.vals, Bp, G, 2)
    for grp in (0, 3):
        for a, b, d in zip(walk, run(A.vals, Bp, G, grp), den):
            assert float(((a - b).abs() - 2 * TOL[torch.float32] * d).max()) <= 0


def test_default_chunks_of_a_wide_panel(shiro):
    """Chunks end at 256 items also where the carry slots then need more than
    the allocation-free product's 32 MiB (the 2^24 panel at N = 256: 34 MB): it
    says so, and runs with chunks of 272."""
    A = synth.config2(device=torch.device("cuda"))
    N = 256
    plan = shiro.partition(A.row_ptr, A.col, A.n_rows, A.n_cols, A.P, A.p)
    U, _ = shiro.select_rows(plan)
    rows = plan.info()["rows"]
    assert shiro.get_tuning(plan, "spmm", N)["chunk"] == 256
    shiro.prepare(plan, N, ops=("spmm",))
    Bp, out = torch.rand(U, N, device="cuda"), torch.empty(rows, N, device="cuda")
    with pytest.raises(shiro.ShiroError) as e:
        shiro.spmm_noalloc(plan, A.vals, Bp, out)
    assert e.value.name == "WORKSPACE"
    shiro.set_tuning(plan, "spmm", N, chunk=272)
    shiro.prepare(plan, N, ops=("spmm",))
    assert torch.equal(shiro.spmm_noalloc(plan, A.vals, Bp, out), shiro.spmm(plan, A.vals, Bp))
