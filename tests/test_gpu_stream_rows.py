"""The row-streaming kernels at the edges of their slices, steps and column blocks.

A row of U^beta^T and the core is cut into slices of 64 packs (128 complex64 or 64
complex128 values), several per wavefront; steps take 1, 2 or 4 rows; up to four
right-hand sides share a sweep.  The layouts below put n_beta at and around whole slices,
the longest row in each kernel (up to 4, 8 or 16 slices a wavefront, and the general
kernels beyond), and r_beta around whole steps.  Bounds: FP32 sums of at most 2e4 products
of O(1 / sqrt(K)) terms in four contractions stay within 1e-5 of the oracle, FP64 within
1e-11.  A pass equals its stages bit for bit.
"""
import numpy as np
import pytest

import synth
from oracle import products as pr
from gpu_util import dev, host, arena, max_rel, l2_rel, banner

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2103_05822_amd")

TOL = {T.FMM_C128: 1e-11, T.FMM_C64: 1e-5}
CDT = {T.FMM_C128: np.complex128, T.FMM_C64: np.complex64}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("prec", [T.FMM_C128, T.FMM_C64], ids=["c128", "c64"])
@pytest.mark.parametrize("longest", [130, 900, 1800, 4100, 9000, 17000])
@pytest.mark.parametrize("threads", [64, 512])
def test_row_slices(prec, longest, threads, monkeypatch):
    monkeypatch.setenv("TUCKFMM_STREAM_THREADS", str(threads))
    sizes = [n for n in (1, 2, 63, 64, 65, 127, 128, 129, 256, 257, 641) if n < longest] + [longest]
    lay = T.Layout(7, 11, np.concatenate([[0], np.cumsum(sizes)]))
    rng = synth.rng(longest)
    tuck = []
    for g, nb in enumerate(sizes):
        pair = []
        for a in range(2):
            rb = min(nb, (1, 2, 3, 4, 5, 8, 9)[(2 * g + a) % 7])
            rt, rp = (7, 11) if g % 3 == 0 else (int(rng.integers(1, 8)), int(rng.integers(1, 12)))
            core, ut, up, ub = synth.synthetic_tucker(rng, 7, 11, nb, rt, rp, rb)
            pair.append((core, (ut, up, ub)))
        tuck.append(pair)
    h = T.fmm_tucker_create(lay)
    try:
        for g, pair in enumerate(tuck):
            for a, (core, (ut, up, ub)) in enumerate(pair):
                T.fmm_tucker_set_group(h, g, a, core, ut, up, ub)
        ar = arena(T.fmm_tucker_storage_bytes(h, prec)[1])
        T.fmm_tucker_upload(h, prec, ar)
        for nrhs in (1, 2, 3, 4, 5):
            banner("row slices prec=%d longest=%d threads=%d nrhs=%d" % (prec, longest, threads, nrhs))
            if not (prec == T.FMM_C128 and longest == 17000):  # that layout runs on the matrix cores
                T.fmm_tucker_set_tuned(h, prec, nrhs, path=0, threads=threads)
            x = synth.complex_normal(rng, (lay.n_basis, nrhs))
            gin = synth.complex_normal(rng, (lay.n_groups, 2, lay.n_dir, nrhs))
            xd, gd = dev(x, CDT[prec]), dev(gin, CDT[prec])
            F, V = dev(np.full(gin.shape, np.nan, CDT[prec])), dev(np.full(x.shape, np.nan, CDT[prec]))
            T.fmm_tucker_pass(h, prec, nrhs, xd, F, gd, V)
            Fp, Vp = host(F).copy(), host(V).copy()
            f_ref = pr.aggregate_all("tucker", tuck, lay.offsets, x)
            v_ref = pr.disaggregate_all("tucker", tuck, lay.offsets, gin)
            errs = (l2_rel(Fp, f_ref), max_rel(Fp, f_ref), l2_rel(Vp, v_ref), max_rel(Vp, v_ref))
            assert max(errs) < TOL[prec], errs
            T.fmm_tucker_aggregate(h, prec, nrhs, xd, F)
            T.fmm_tucker_disaggregate(h, prec, nrhs, gd, V)
            assert np.array_equal(host(F), Fp) and np.array_equal(host(V), Vp)
    finally:
        T.fmm_tucker_destroy(h)
