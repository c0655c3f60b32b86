"""Layouts with an item beyond the streaming kernels' LDS: an even number of right-hand sides
runs on the matrix cores in every precision, 2 and 4 included; an odd one is refused in
complex64 (FMM_ERR_UNSUPPORTED) and runs on the matrix cores in complex128.  Bounds: 1e-11
(FP64) and 1e-5 (FP32) against the oracle.
"""
import numpy as np
import pytest

import synth
from oracle import products as pr
from gpu_util import dev, host, arena, l2_rel, banner

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2103_05822_amd")

TOL = {T.FMM_C128: 1e-11, T.FMM_C64: 1e-5}
CDT = {T.FMM_C128: np.complex128, T.FMM_C64: np.complex64}


@pytest.mark.parametrize("prec", [T.FMM_C128, T.FMM_C64], ids=["c128", "c64"])
def test_item_beyond_lds(prec):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    sizes = [21000, 40, 3]
    lay = T.Layout(5, 9, np.concatenate([[0], np.cumsum(sizes)]))
    rng = synth.rng(3)
    tuck = []
    for nb in sizes:
        pair = []
        for _ in range(2):
            core, ut, up, ub = synth.synthetic_tucker(rng, 5, 9, nb, 3, 3, 3)
            pair.append((core, (ut, up, ub)))
        tuck.append(pair)
    h = T.fmm_tucker_create(lay)
    try:
        for g, pair in enumerate(tuck):
            for a, (core, (ut, up, ub)) in enumerate(pair):
                T.fmm_tucker_set_group(h, g, a, core, ut, up, ub)
        ar = arena(T.fmm_tucker_storage_bytes(h, prec)[1])
        T.fmm_tucker_upload(h, prec, ar)
        for nrhs in (1, 2, 3, 4, 6):
            banner("large item prec=%d nrhs=%d" % (prec, nrhs))
            x = synth.complex_normal(rng, (lay.n_basis, nrhs))
            gin = synth.complex_normal(rng, (lay.n_groups, 2, lay.n_dir, nrhs))
            xd, gd = dev(x, CDT[prec]), dev(gin, CDT[prec])
            F, V = torch.zeros_like(gd), torch.zeros_like(xd)
            if prec == T.FMM_C64 and nrhs % 2:
                with pytest.raises(T.FmmError) as e:
                    T.fmm_tucker_pass(h, prec, nrhs, xd, F, gd, V)
                assert e.value.status == -6
                continue
            T.fmm_tucker_pass(h, prec, nrhs, xd, F, gd, V)
            assert l2_rel(host(F), pr.aggregate_all("tucker", tuck, lay.offsets, x)) < TOL[prec]
            assert l2_rel(host(V), pr.disaggregate_all("tucker", tuck, lay.offsets, gin)) < TOL[prec]
    finally:
        T.fmm_tucker_destroy(h)
