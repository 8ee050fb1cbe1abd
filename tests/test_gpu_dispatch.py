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
