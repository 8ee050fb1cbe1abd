"""The nonzero walk at the edges of its tiles: widths around its 64-lane
columns-per-lane steps, ragged and odd widths, rows that are no whole dwords
(the 64-bit gather), chunks that cut rows into many pieces, hub and empty
rows, several column tiles with their partial dots."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

# componentwise against |A||B|: float32 sums of at most a few hundred terms,
# bfloat16 inputs and outputs rounded once each (2^-8 relative per rounding)
TOL = {torch.float32: 1e-5, torch.bfloat16: 1e-2}


@pytest.fixture(scope="module")
def shiro():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_20178_amd as s

    s._lib.load()
    return s


def _case(seed):
    rng = np.random.default_rng(seed)
    rows, cols = 150, 333
    mask = rng.random((rows, cols)) < 0.04
    mask[40, :] = rng.random(cols) < 0.8  # cut by many chunks
    mask[60:75, :] = False  # empty rows inside a chunk
    mask[-1, :] = False
    vals = rng.uniform(0.1, 1, size=(rows, cols)).astype(np.float32) * mask
    return synth.from_dense_pattern(vals, P=1, p=0, name="walk")


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N", [1, 2, 31, 63, 64, 65, 127, 128, 129, 193, 257, 513])
def test_walk_tile_edges(shiro, N, dtype):
    A = _case(N)
    dev = torch.device("cuda")
    Ad, Ac = A.to(dev), oracle.Csr.from_synth(A)
    plan = shiro.partition(Ad.row_ptr, Ad.col, A.n_rows, A.n_cols, 1, 0, check=True)
    U, _ = shiro.select_rows(plan)
    B = synth.dense(A.n_cols, N, N, synth.STREAM_B).to(dtype)
    G = synth.dense(A.n_rows, N, N, synth.STREAM_DY).to(dtype)
    Bn, Gn = B.float().numpy(), G.float().numpy()
    tol = TOL[dtype]
    Y0 = oracle.spmm(Ac, Bn, None), oracle.spmm(Ac, Bn, None, abs_mode=True)
    uc, _, cm = oracle.select(Ac)
    dB0 = oracle.spmm_t(Ac, Gn, cm, n_out=U), oracle.spmm_t(Ac, Gn, cm, n_out=U, abs_mode=True)
    dv0 = oracle.sddmm(Ac, Gn, Bn, None), oracle.sddmm(Ac, Gn, Bn, None, abs_mode=True)
    for chunk, lanes, pad in ((16, 64, 0), (100, 16, 1), (4096, 32, 3)):
        for k in ("spmm", "spmm_t"):
            shiro.set_tuning(plan, k, N, dtype, chunk=chunk, lanes=lanes, group_rows=2)
        Bd = torch.zeros(A.n_cols, N + pad, dtype=dtype, device=dev)[:, :N].copy_(B)
        Gd = torch.zeros(A.n_rows, N + pad, dtype=dtype, device=dev)[:, :N].copy_(G)
        Bp = shiro.pack_B(plan, Bd, out=torch.empty(U, N + pad, dtype=dtype, device=dev)[:, :N])
        Y = torch.full((A.n_rows, N + pad), float("nan"), dtype=dtype, device=dev)[:, :N]
        shiro.spmm(plan, Ad.vals, Bp, out=Y)
        assert oracle.rel_err(Y.float().cpu().numpy(), *Y0) <= tol, (chunk, lanes, pad)
        dBp = torch.full((U, N + pad), float("nan"), dtype=dtype, device=dev)[:, :N]
        dB = torch.ones(A.n_cols, N, dtype=dtype, device=dev)  # rows added to, every column once
        dvals = torch.zeros(A.nnz, device=dev)
        shiro.spmm_backward(plan, Ad.vals, Gd, Bp, dBpacked=dBp, dB=dB, dvals=dvals)
        assert oracle.rel_err(dBp.float().cpu().numpy(), *dB0) <= tol, (chunk, lanes, pad)
        full, fden = np.ones((A.n_cols, N)), np.ones((A.n_cols, N))
        full[uc] += dB0[0]
        fden[uc] += dB0[1]
        assert oracle.rel_err(dB.float().cpu().numpy(), full, fden) <= tol, (chunk, lanes, pad)
        assert oracle.rel_err(dvals.cpu().numpy(), *dv0) <= TOL[torch.float32], (chunk, lanes, pad)


@pytest.mark.parametrize("N", [1, 32, 256, 1024])
def test_default_chunks(shiro, N):
    """Default chunks: 16 to 256 items, at most 16384 chunks unless they have
    256 items, and no more carry slots than the allocation-free product holds
    where 256-item chunks fit it; the product through it equals spmm."""
    A = synth.small_rmat(13, 16)
    dev = torch.device("cuda")
    Ad = A.to(dev)
    plan = shiro.partition(Ad.row_ptr, Ad.col, A.n_rows, A.n_cols, 1, 0)
    U, _ = shiro.select_rows(plan)
    items = A.n_rows + A.nnz
    for k in ("spmm", "spmm_t"):
        c = shiro.get_tuning(plan, k, N)["chunk"]
        n = -(-(items if k == "spmm" else U + A.nnz) // c)
        assert 16 <= c <= 256 and (c == 256 or (n <= 16384 and 2 * n * N * 4 <= 32 << 20))
    shiro.prepare(plan, N, ops=("spmm",))
    Bp = synth.dense(U, N, 0, synth.STREAM_B).to(dev)
    out = torch.empty(A.n_rows, N, device=dev)
    assert torch.equal(shiro.spmm_noalloc(plan, Ad.vals, Bp, out), shiro.spmm(plan, Ad.vals, Bp))


@pytest.mark.parametrize("n_rows", [1 << 19, 1 << 18])
def test_staged_value_permutation(shiro, n_rows):
    """Values in and gradients out of the transposed order through the staged
    order of large patterns (13M nonzeros; the smaller pattern, 6.5M, keeps the
    direct permutation).  One nonzero value per row and column id makes every
    moved value visible: dB[c] = sum of the values of column c, dvals[k] = the
    product of two small integers, both exact in float32."""
    dev = torch.device("cuda")
    deg = 25
    g = torch.Generator(device=dev)
    g.manual_seed(n_rows)
    # deg distinct columns per row, ascending
    step = n_rows // deg
    col = torch.randint(step, (n_rows, deg), generator=g, device=dev) + torch.arange(deg, device=dev) * step
    row_ptr = torch.arange(0, n_rows * deg + 1, deg, device=dev)
    vals = torch.randint(-3, 4, (n_rows * deg,), generator=g, device=dev).float()
    plan = shiro.partition(row_ptr, col.reshape(-1).int(), n_rows, n_rows, 1, 0)
    U, _ = shiro.select_rows(plan)
    G = torch.randint(-2, 3, (n_rows, 1), generator=g, device=dev).float()
    B = torch.randint(-2, 3, (n_rows, 1), generator=g, device=dev).float()
    Bp = shiro.pack_B(plan, B)
    dB = torch.zeros_like(B)
    dvals = torch.full_like(vals, float("nan"))
    shiro.spmm_backward(plan, vals, G, Bp, dB=dB, dvals=dvals, dB_overwrite=True)
    rows = torch.arange(n_rows, device=dev).repeat_interleave(deg)
    want = torch.zeros(n_rows, dtype=torch.float64, device=dev)
    want.index_add_(0, col.reshape(-1), (vals * G[rows, 0]).double())
    assert torch.equal(dB[:, 0].double(), want)
    assert torch.equal(dvals, G[rows, 0] * B[col.reshape(-1), 0])


@pytest.mark.parametrize("P,p", [(1, 0), (4, 1)])
def test_autograd_gradients_complete(shiro, P, p):
    """Gradients that the backward writes whole are not zero-filled first; the
    others are: stale memory never shows, a panel's gradients are zero outside
    it."""
    A = synth.small_rmat(9, 40, P=P, p=p)
    dev = torch.device("cuda")
    Ad, Ac = A.to(dev), oracle.Csr.from_synth(A)
    plan = shiro.partition(Ad.row_ptr, Ad.col, A.n_rows, A.n_cols, P, p)
    shiro.select_rows(plan)
    N = 16
    B = synth.dense(A.n_cols, N, 0, synth.STREAM_B).to(dev)
    G = synth.dense(plan.info()["rows"], N, 0, synth.STREAM_DY).to(dev)
    for t in (A.nnz, A.n_cols * N):  # what the allocator hands out next holds NaN
        stale = [torch.full((t,), float("nan"), device=dev) for _ in range(4)]
        del stale
    vals, Bl = Ad.vals.clone().requires_grad_(True), B.clone().requires_grad_(True)
    Y = shiro.shiro_spmm(plan, vals, Bl)
    dvals, dB = torch.autograd.grad(Y, (vals, Bl), G)
    Bn, Gn = B.cpu().numpy(), G.cpu().numpy()
    assert oracle.rel_err(dB.cpu().numpy(), oracle.spmm_t(Ac, Gn, None), oracle.spmm_t(Ac, Gn, None, abs_mode=True)) <= 1e-5
    nz = slice(Ac.nz_begin, Ac.nz_begin + Ac.nnz_panel)
    dv = dvals.cpu().numpy()
    assert oracle.rel_err(dv[nz], oracle.sddmm(Ac, Gn, Bn, None), oracle.sddmm(Ac, Gn, Bn, None, abs_mode=True)) <= 1e-5
    rest = np.delete(dv, np.arange(A.nnz)[nz])
    assert not rest.any()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N", [3, 4, 5, 31, 32, 33, 47, 63, 64, 65, 130])
def test_value_gradients_alone(shiro, N, dtype):
    """dvals without dB at the width edges of its kernels (lane groups of 8 and
    16 from 4 to 64 columns, the walk outside), padded rows, and a nonzero
    count that is no whole number of windows."""
    A = _case(100 + N)
    dev = torch.device("cuda")
    Ad, Ac = A.to(dev), oracle.Csr.from_synth(A)
    plan = shiro.partition(Ad.row_ptr, Ad.col, A.n_rows, A.n_cols, 1, 0)
    U, _ = shiro.select_rows(plan)
    B = synth.dense(A.n_cols, N, N, synth.STREAM_B).to(dtype)
    G = synth.dense(A.n_rows, N, N, synth.STREAM_DY).to(dtype)
    Bn, Gn = B.float().numpy(), G.float().numpy()
    ref, den = oracle.sddmm(Ac, Gn, Bn, None), oracle.sddmm(Ac, Gn, Bn, None, abs_mode=True)
    for pad in (0, 1):
        Bp = shiro.pack_B(plan, B.to(dev), out=torch.empty(U, N + pad, dtype=dtype, device=dev)[:, :N])
        Gd = torch.zeros(A.n_rows, N + pad, dtype=dtype, device=dev)[:, :N].copy_(G)
        dvals = torch.full((A.nnz,), float("nan"), device=dev)
        shiro.spmm_backward(plan, None, Gd, Bp, dvals=dvals)
        assert oracle.rel_err(dvals.cpu().numpy(), ref, den) <= 1e-5, pad
