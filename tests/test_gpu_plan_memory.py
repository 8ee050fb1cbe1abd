"""Device memory of a plan: what preparing it allocates, what happens when an
allocation fails part way, and that no buffer a captured graph may hold is
given back while the plan lives.  A counting allocator (torch tensors) stands
behind the library in every test."""
import contextlib

import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def shiro():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_20178_amd as s

    s._lib.load()
    return s


_HOOKS = []


class Arena:
    """refuse(bytes) true: no memory for that request."""

    def __init__(self):
        self.live, self.freed, self.asked = {}, [], []
        self.refuse = lambda n: False

    def held(self):
        return sum(t.numel() for t in self.live.values())

    def alloc(self, n, ctx):
        self.asked.append(int(n))
        if self.refuse(int(n)):
            return None
        t = torch.empty(int(n), dtype=torch.uint8, device="cuda")
        self.live[t.data_ptr()] = t
        return t.data_ptr()

    def free(self, p, n, ctx):
        self.freed.append(p)
        self.live.pop(p)


@contextlib.contextmanager
def arena(shiro):
    a = Arena()
    hooks = (shiro._lib.ALLOC_FN(a.alloc), shiro._lib.FREE_FN(a.free))
    _HOOKS.append(hooks)  # outlive any plan a failing test leaves behind
    assert shiro._L().shiro_set_allocator(hooks[0], hooks[1], None) == 0
    try:
        yield a
    finally:
        shiro.use_torch_allocator(False)


def _backward(shiro, plan, vals, N, dtype=torch.float32):
    dev = vals.device
    inf = plan.info()
    Bp = synth.dense(inf["U"], N, 1, synth.STREAM_B).to(dev).to(dtype)
    G = synth.dense(inf["rows"], N, 2, synth.STREAM_DY).to(dev).to(dtype)
    dBp = torch.full((inf["U"], N), float("nan"), dtype=dtype, device=dev)
    dvals = torch.full_like(vals, float("nan"))
    shiro.spmm_backward(plan, vals, G, Bp, dBpacked=dBp, dvals=dvals)
    return dBp, dvals


def test_failed_allocation_leaves_nothing_behind(shiro):
    """Each allocation of prepare fails once: the call reports OOM, a second
    call succeeds with the same results, and the plan gives back every block
    when it is destroyed."""
    A, N = synth.small_rmat(10, 16), 32
    Ad = A.to(torch.device("cuda"))
    plan = shiro.partition(Ad.row_ptr, Ad.col, A.n_rows, A.n_cols, 1, 0)
    shiro.select_rows(plan)
    want = _backward(shiro, plan, Ad.vals, N)
    failures = 0
    with arena(shiro) as a:
        for k in range(100):
            plan = shiro.partition(Ad.row_ptr, Ad.col, A.n_rows, A.n_cols, 1, 0)
            shiro.select_rows(plan)
            last = len(a.asked) + k + 1
            a.refuse = lambda n: len(a.asked) == last
            try:
                shiro.prepare(plan, N)
                done = len(a.asked) < last
            except shiro.ShiroError as e:
                assert e.name == "OOM"
                done, failures = False, failures + 1
            a.refuse = lambda n: False
            shiro.prepare(plan, N)
            got = _backward(shiro, plan, Ad.vals, N)
            plan.close()
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), k
            assert not a.live, f"allocation {k}: {len(a.live)} blocks not given back"
            if done:
                break
    assert done and failures >= 8


def _large(n_rows=1 << 19, deg=25):
    """13.1M nonzeros, deg ascending columns a row; small whole numbers, so
    every gradient at N = 1 is exact."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(7)
    step = n_rows // deg
    col = torch.randint(step, (n_rows, deg), generator=g, device=dev) + torch.arange(deg, device=dev) * step
    row_ptr = torch.arange(0, n_rows * deg + 1, deg, device=dev)
    vals = torch.randint(-3, 4, (n_rows * deg,), generator=g, device=dev).float()
    G = torch.randint(-2, 3, (n_rows, 1), generator=g, device=dev).float()
    B = torch.randint(-2, 3, (n_rows, 1), generator=g, device=dev).float()
    return row_ptr, col, vals, G, B


def _check_large(shiro, plan, case):
    row_ptr, col, vals, G, B = case
    n_rows, deg = col.shape
    Bp = shiro.pack_B(plan, B)
    dB = torch.zeros_like(B)
    dvals = torch.full_like(vals, float("nan"))
    shiro.spmm_backward(plan, vals, G, Bp, dB=dB, dvals=dvals, dB_overwrite=True)
    rows = torch.arange(n_rows, device=vals.device).repeat_interleave(deg)
    want = torch.zeros(n_rows, dtype=torch.float64, device=vals.device)
    want.index_add_(0, col.reshape(-1), (vals * G[rows, 0]).double())
    assert torch.equal(dB[:, 0].double(), want)
    assert torch.equal(dvals, G[rows, 0] * B[col.reshape(-1), 0])


def test_large_pattern_without_memory_for_the_staged_order(shiro):
    """The staged value order is an optimisation: with memory for the direct
    permutation only (row ids, the transposed pattern's three arrays, values
    and gradients: 24 bytes a nonzero beside the work lists) prepare succeeds
    and the gradients are the same."""
    case = _large()
    row_ptr, col, vals, _, _ = case
    n, nnz = col.shape[0], vals.numel()
    with arena(shiro) as a:
        plan = shiro.partition(row_ptr, col.reshape(-1).int(), n, n, 1, 0)
        shiro.select_rows(plan)
        limit = a.held() + 24 * nnz + 8 * n + (16 << 20)
        a.refuse = lambda b: a.held() + b > limit
        shiro.prepare(plan, 1)
        _check_large(shiro, plan, case)
        plan.close()
        assert not a.live


def test_large_pattern_setup_memory(shiro):
    """Preparing a pattern in the staged order allocates one array (4 bytes a
    nonzero) more than the direct permutation needs, gives no large block back
    and allocates none twice."""
    case = _large()
    row_ptr, col, vals, _, _ = case
    n, nnz = col.shape[0], vals.numel()
    with arena(shiro) as a:
        plan = shiro.partition(row_ptr, col.reshape(-1).int(), n, n, 1, 0)
        shiro.select_rows(plan)
        first = len(a.asked)
        before = dict(a.live)
        shiro.prepare(plan, 1)
        big = [b for b in a.asked[first:] if b >= 2 * nnz]
        assert sum(a.asked[first:]) <= 28 * nnz + 8 * n + (16 << 20)
        assert len(big) == 7
        assert all(p in a.live for p in before)
        _check_large(shiro, plan, case)
        plan.close()
        assert not a.live


def test_several_tiles_without_memory_for_their_gradients(shiro):
    """dvals over several column tiles keep one set of partial sums per tile;
    with memory for one set only, the product and the value gradients run as
    two passes instead of failing."""
    A, N = synth.small_rmat(12, 16), 320
    Ad = A.to(torch.device("cuda"))
    plan = shiro.partition(Ad.row_ptr, Ad.col, A.n_rows, A.n_cols, 1, 0)
    shiro.select_rows(plan)
    want = _backward(shiro, plan, Ad.vals, N)
    one = 4 * plan.info()["nnz"]
    with arena(shiro) as a:
        a.refuse = lambda b: b in (2 * one, 3 * one, 4 * one)
        plan = shiro.partition(Ad.row_ptr, Ad.col, A.n_rows, A.n_cols, 1, 0)
        shiro.select_rows(plan)
        shiro.prepare(plan, N)
        got = _backward(shiro, plan, Ad.vals, N)
        plan.close()
        assert not a.live
    assert torch.equal(got[0], want[0])
    # float32 dots of 320 terms, componentwise against |dY||B|
    Bp = synth.dense(len(want[0]), N, 1, synth.STREAM_B).numpy()
    G = synth.dense(A.n_rows, N, 2, synth.STREAM_DY).numpy()
    Ac = oracle.Csr.from_synth(A)
    cm = oracle.select(Ac)[2]
    ref, den = oracle.sddmm(Ac, G, Bp, cm), oracle.sddmm(Ac, G, Bp, cm, abs_mode=True)
    for dv in (want[1], got[1]):
        assert oracle.rel_err(dv.cpu().numpy(), ref, den) <= 1e-5


def test_buffers_of_a_captured_graph_stay(shiro):
    """A graph captured by the caller (not by the library) holds the plan's
    buffers by address.  Later calls that need larger ones leave those alone,
    and the replay still gives the captured call's results."""
    A, N = synth.small_rmat(11, 16), 130
    dev = torch.device("cuda")
    Ad = A.to(dev)
    with arena(shiro) as a:
        plan = shiro.partition(Ad.row_ptr, Ad.col, A.n_rows, A.n_cols, 1, 0)
        U, _ = shiro.select_rows(plan)
        shiro.prepare(plan, N)
        Bp = synth.dense(U, N, 1, synth.STREAM_B).to(dev)
        G = synth.dense(A.n_rows, N, 2, synth.STREAM_DY).to(dev)
        Y = torch.empty(A.n_rows, N, device=dev)
        dBp, dvals = torch.empty(U, N, device=dev), torch.empty(A.nnz, device=dev)

        def step():
            shiro.spmm(plan, Ad.vals, Bp, out=Y)
            shiro.spmm_backward(plan, Ad.vals, G, Bp, dBpacked=dBp, dvals=dvals)

        step()
        torch.cuda.synchronize()
        want = [t.clone() for t in (Y, dBp, dvals)]
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step()
        torch.cuda.synchronize()
        at_capture = set(a.live)
        for wider in (260, 520):  # larger carry slots, more sets of partial dots
            shiro.prepare(plan, wider)
            _backward(shiro, plan, Ad.vals, wider)
        torch.cuda.synchronize()
        gone = at_capture - set(a.live)
        assert not gone, f"{len(gone)} blocks given back under a captured graph"
        for _ in range(3):
            for t in (Y, dBp, dvals):
                t.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            for t, w in zip((Y, dBp, dvals), want):
                assert torch.equal(t, w)
            _backward(shiro, plan, Ad.vals, 64)  # eager work between the replays
        del graph
        plan.close()
        assert not a.live


def test_launch_errors_of_subset_plans_are_reported(shiro):
    """An error the runtime holds when a product is launched is reported by
    the call, on plans that gather their values first as on the others."""
    import ctypes

    A, N = synth.small_rmat(8, 8), 16
    dev = torch.device("cuda")
    Ad = A.to(dev)
    hip = ctypes.CDLL("libamdhip64.so")
    L = shiro._L()
    keep = torch.ones(A.nnz, dtype=torch.uint8, device=dev)
    codes = []
    for subset in (False, True):
        if subset:
            plan = shiro.partition_subset(Ad.row_ptr, Ad.col, A.n_rows, A.n_cols, 1, 0, keep, 1)
        else:
            plan = shiro.partition(Ad.row_ptr, Ad.col, A.n_rows, A.n_cols, 1, 0)
        U, _ = shiro.select_rows(plan)
        shiro.prepare(plan, N)
        Bp = synth.dense(U, N, 1, synth.STREAM_B).to(dev)
        Y = torch.empty(A.n_rows, N, device=dev)
        args = (plan.handle, Ad.vals.data_ptr(), Bp.data_ptr(), N, N, shiro._lib.F32, Y.data_ptr(), N,
                shiro._lib.F32, shiro._lib.MODE_BATCHED, shiro._stream())
        torch.cuda.synchronize()
        assert L.shiro_spmm(*args) == 0
        torch.cuda.synchronize()
        assert hip.hipSetDevice(9999) != 0  # leaves an error for the next check
        codes.append(L.shiro_spmm(*args))
        hip.hipGetLastError()
        torch.cuda.synchronize()
        plan.close()
    assert codes[0] == codes[1]


@pytest.mark.parametrize("N", [32, 130, 256])
def test_prepare_gives_nothing_back(shiro, N):
    """Preparing a plan's product and backward allocates what stays and nothing
    else: no temporary blocks, no buffer that a later step of it replaces."""
    A = synth.small_rmat(13, 16)
    Ad = A.to(torch.device("cuda"))
    with arena(shiro) as a:
        plan = shiro.partition(Ad.row_ptr, Ad.col, A.n_rows, A.n_cols, 1, 0)
        shiro.select_rows(plan)
        before = len(a.freed)
        shiro.prepare(plan, N)
        assert len(a.freed) == before
        _backward(shiro, plan, Ad.vals, N)
        assert len(a.freed) == before
        plan.close()
        assert not a.live


def test_whole_plan_memory(shiro):
    """A plan of 13M nonzeros, from partition to the prepared backward: 49 bytes
    a nonzero (column ids three times, 9 of sort scratch, the transposed
    pattern, row ids, values and gradients, the staged order) beside the row
    and column arrays, work lists and carry slots."""
    case = _large()
    row_ptr, col, vals, _, _ = case
    n, nnz = col.shape[0], vals.numel()
    with arena(shiro) as a:
        plan = shiro.partition(row_ptr, col.reshape(-1).int(), n, n, 1, 0)
        shiro.select_rows(plan)
        shiro.prepare(plan, 1)
        assert sum(a.asked) <= 50 * nnz + 32 * n + (16 << 20)
        _check_large(shiro, plan, case)
        plan.close()
        assert not a.live
