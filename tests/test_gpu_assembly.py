"""X from its factors, entry by entry against FP64: whole blocks of 64 x 64 and ragged ones, ranks about the chunk of 16.

A component of an entry is a chain of 2 k FP32 fused multiply-adds, so its error is at most 2 k u sum |l_k| |r_k|
(u = 2^-24, |ac| + |bd| <= |l| |r|); two components, and one rounding of theta and of the result: sqrt(2) (2 k + 2) u.
"""
import numpy as np
import pytest

import oracle as O
import synth
from gpu_cases import from_geometry, to_device

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("grid,tiles,k_off,k_diag", [
    ((16, 8), [64, 64], 16, 17),          # whole blocks, one chunk and one entry more
    ((16, 16), [128, 128], 33, 48),       # blocks below, on and right of a diagonal tile's block diagonal
    ((23, 7), [65, 65, 31], 15, 1),       # a row and a column past a block
    ((20, 13), [130, 130], 32, -1),       # two of them, dense diagonals
    ((9, 7), [63], 1, 31),                # one block, not whole
])
def test_entries(grid, tiles, k_off, k_diag):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2412_14973_amd as tl
    nt = len(tiles)
    lay = synth.Layout(np.array(tiles), np.full(nt * (nt - 1) // 2, k_off), np.full(nt, k_diag))
    case = from_geometry(*grid, "half", 12.0, lay, 91, "entries")
    plan, D, U, th, _ = to_device(case, tl, torch)
    X = tl.forward(plan, D, U, th, want_X=True)[-1].cpu().numpy().astype(np.complex128)
    bound = np.sqrt(2) * (2 * max(k_off, k_diag) + 2) * 2.0 ** -24 * O.assemble(case.T, np.abs(case.theta).astype(complex)).real
    err = np.abs(X - O.assemble(case.T, case.theta))
    print(f"largest error over its bound {np.max(err / bound):.2e}")
    assert np.all(err <= bound)
    assert np.array_equal(X, X.T)
