"""The dense aggregation with 2 to 5 right-hand sides on both sides of its row limits.

Groups of at most 24 mean rows in complex128, in complex64 of 40 (2 right-hand sides) or 20,
with more than 128 columns run on the vector units, others and more right-hand sides on the
matrix cores.  Sums of at most 45 products: 1e-13 (FP64) and 1e-5 (FP32) against the sums'
definition.  The columns sit around 128 and the 512 of a workgroup.
"""
import numpy as np
import pytest

import synth
from gpu_util import dev, host, max_rel, banner

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2103_05822_amd")

TOL = {T.FMM_C128: 1e-13, T.FMM_C64: 1e-5}
CDT = {T.FMM_C128: np.complex128, T.FMM_C64: np.complex64}


@pytest.mark.parametrize("prec", [T.FMM_C128, T.FMM_C64], ids=["c128", "c64"])
@pytest.mark.parametrize("grid", [(1, 1), (8, 8), (8, 9), (15, 17), (16, 16), (3, 86)])
@pytest.mark.parametrize("rows", [1, 2, 5, 20, 21, 24, 25, 40, 41])
def test_aggregation_of_few_rows(prec, grid, rows):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sizes = [max(1, rows - 4), rows, rows + min(4, rows - 1)]  # mean `rows`
    lay = T.Layout(grid[0], grid[1], np.concatenate([[0], np.cumsum(sizes)]))
    rng = synth.rng(7 * rows + grid[1])
    A = synth.complex_normal(rng, (lay.n_basis, 2, lay.n_dir))
    d = T.fmm_dense_create(lay)
    try:
        Ad = dev(A, CDT[prec])
        for nrhs in (2, 3, 4, 5):
            banner("dense few prec=%d grid=%s rows=%d nrhs=%d" % (prec, grid, rows, nrhs))
            x = synth.complex_normal(rng, (lay.n_basis, nrhs))
            F = dev(np.full((lay.n_groups, 2, lay.n_dir, nrhs), np.nan, CDT[prec]))
            T.fmm_dense_aggregate(d, prec, Ad, nrhs, dev(x, CDT[prec]), F)
            ref = np.stack([np.tensordot(A[a:b], x[a:b], axes=(0, 0)) for a, b in zip(lay.offsets[:-1], lay.offsets[1:])])
            assert max_rel(host(F), ref) < TOL[prec]
    finally:
        T.fmm_dense_destroy(d)
