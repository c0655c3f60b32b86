"""Matrix-core tiles of few rows, whose wavefronts split the columns instead of the rows.

The split changes at 16, 32 and 48 rows left in a tile and at 16 and 32 columns; r_beta,
the angular ranks and the grid below sit on both sides of each, with chunk widths around 16,
32 and 64 right-hand sides.  Bounds as for the path's other shapes: 1e-11 (FP64), 1e-5
(FP32 and the three-piece split) and, for the two-piece split, whose products carry 2^-16
each, 3e-5 in the 2-norm.  A pass equals its stages bit for bit.
"""
import numpy as np
import pytest

import synth
from oracle import products as pr
from gpu_util import dev, host, arena, l2_rel, banner

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2103_05822_amd")

TOL = {T.FMM_C128: 1e-11, T.FMM_C64: 1e-5, T.FMM_BF16X3: 1e-5, T.FMM_BF16X2: 3e-5}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("prec", list(TOL), ids=["c128", "c64", "bf16x3", "bf16x2"])
@pytest.mark.parametrize("nrhs", [8, 16, 18, 32, 34, 64, 66])
def test_column_split_tiles(prec, nrhs):
    ranks = [1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 81, 113]
    sizes = [r + (i % 3) for i, r in enumerate(ranks)]
    lay = T.Layout(49, 33, np.concatenate([[0], np.cumsum(sizes)]))
    rng = synth.rng(500 + nrhs)
    tuck = []
    for g, nb in enumerate(sizes):
        pair = []
        for a in range(2):
            rt, rp = min(49, ranks[(g + a) % 10]), min(33, ranks[(g + 3 * a) % 7])
            core, ut, up, ub = synth.synthetic_tucker(rng, 49, 33, nb, rt, rp, ranks[g])
            pair.append((core, (ut, up, ub)))
        tuck.append(pair)
    cd = np.complex128 if prec == T.FMM_C128 else np.complex64
    h = T.fmm_tucker_create(lay)
    try:
        for g, pair in enumerate(tuck):
            for a, (core, (ut, up, ub)) in enumerate(pair):
                T.fmm_tucker_set_group(h, g, a, core, ut, up, ub)
        ar = arena(T.fmm_tucker_storage_bytes(h, prec)[1])
        T.fmm_tucker_upload(h, prec, ar)
        x = synth.complex_normal(rng, (lay.n_basis, nrhs))
        gin = synth.complex_normal(rng, (lay.n_groups, 2, lay.n_dir, nrhs))
        f_ref = pr.aggregate_all("tucker", tuck, lay.offsets, x)
        v_ref = pr.disaggregate_all("tucker", tuck, lay.offsets, gin)
        xd, gd = dev(x, cd), dev(gin, cd)
        for order in (1, 2):
            banner("column split prec=%d nrhs=%d order=%d" % (prec, nrhs, order))
            T.fmm_tucker_set_tuned(h, prec, nrhs, path=1, tile_steps=16, rhs_chunk=nrhs, order=order)
            F, V = dev(np.full(gin.shape, np.nan, cd)), dev(np.full(x.shape, np.nan, cd))
            T.fmm_tucker_pass(h, prec, nrhs, xd, F, gd, V)
            Fp, Vp = host(F).copy(), host(V).copy()
            errs = (l2_rel(Fp, f_ref), l2_rel(Vp, v_ref))
            assert max(errs) < TOL[prec], errs
            T.fmm_tucker_aggregate(h, prec, nrhs, xd, F)
            T.fmm_tucker_disaggregate(h, prec, nrhs, gd, V)
            assert np.array_equal(host(F), Fp) and np.array_equal(host(V), Vp)
    finally:
        T.fmm_tucker_destroy(h)
