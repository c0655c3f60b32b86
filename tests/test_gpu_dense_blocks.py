"""The dense kernels at the edges of their blocks: rows around the 16 of a row block, the 4
of a step and the wavefronts' turns, columns around the 64 of a workgroup and the 4 of a
step, right-hand sides around the 8 that share a read.  Bounds: sums of at most 260 products
in FP64 (1e-13) and FP32 (1e-5) against the oracle.
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
@pytest.mark.parametrize("grid", [(1, 1), (3, 5), (7, 9), (8, 8), (5, 13), (10, 13)])
def test_dense_block_edges(prec, grid):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sizes = [1, 2, 3, 4, 5, 13, 15, 16, 17, 31, 32, 33, 65, 130]
    lay = T.Layout(grid[0], grid[1], np.concatenate([[0], np.cumsum(sizes)]))
    rng = synth.rng(10 * grid[0] + grid[1])
    A = synth.complex_normal(rng, (lay.n_basis, 2, lay.n_dir))
    d = T.fmm_dense_create(lay)
    try:
        Ad = dev(A, CDT[prec])
        for nrhs in (1, 2, 3, 7, 8, 9, 17):
            banner("dense blocks prec=%d grid=%s nrhs=%d" % (prec, grid, nrhs))
            x = synth.complex_normal(rng, (lay.n_basis, nrhs))
            gin = synth.complex_normal(rng, (lay.n_groups, 2, lay.n_dir, nrhs))
            F, V = dev(np.full(gin.shape, np.nan, CDT[prec])), dev(np.full(x.shape, np.nan, CDT[prec]))
            T.fmm_dense_aggregate(d, prec, Ad, nrhs, dev(x, CDT[prec]), F)
            T.fmm_dense_disaggregate(d, prec, Ad, nrhs, dev(gin, CDT[prec]), V)
            blocks = [A[lay.offsets[g]:lay.offsets[g + 1]] for g in range(lay.n_groups)]
            f_ref = np.stack([np.einsum("nad,nr->adr", b, x[lay.offsets[g]:lay.offsets[g + 1]])
                              for g, b in enumerate(blocks)])
            v_ref = np.concatenate([np.einsum("nad,adr->nr", b.conj(), gin[g]) for g, b in enumerate(blocks)])
            assert max_rel(host(F), f_ref) < TOL[prec] and max_rel(host(V), v_ref) < TOL[prec]
    finally:
        T.fmm_dense_destroy(d)
