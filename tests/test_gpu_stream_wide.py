"""The row-streaming kernels at every number of slices a wavefront holds, with and without row
blocks.

A row of U^beta^T and the core is cut into slices of 64 packs (128 complex64 or 64 complex128
values); the wavefronts of a workgroup share them.  The layouts hold an item for every number
of slices a wavefront from 1 to the largest of a kernel (4, 8, or 12 with 512 threads; with 13 the
general kernel runs the layout), its last slice partly filled.  `split` cuts the items into row blocks whose partial sums are added
afterwards.  Bounds: FP32 sums of at most 2e4 products of O(1 / sqrt(K)) terms in four
contractions within 1e-5 of the oracle, FP64 within 1e-11.  A pass equals its stages bit for bit.
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
NT, NP = 7, 11  # a core row of at most 77 values: one slice (complex64) or two


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


def _slices(prec, nb, q):
    E = 2 if prec == T.FMM_C64 else 1
    packs = lambda n: -(-n // E)  # noqa: E731
    return -(-packs(nb) // 64) + -(-packs(q) // 64)


@pytest.mark.parametrize("prec", [T.FMM_C128, T.FMM_C64], ids=["c128", "c64"])
@pytest.mark.parametrize("threads,most", [(64, 4), (64, 8), (128, 4), (128, 8), (256, 8), (512, 4), (512, 8), (512, 12), (512, 13)])
@pytest.mark.parametrize("split", [False, True])
def test_slices_per_wavefront(prec, threads, most, split, monkeypatch):
    if split:
        monkeypatch.setenv("TUCKFMM_SPLIT_ELEMS", "2000")
    E, nw, rt, rp = (2 if prec == T.FMM_C64 else 1), threads // 64, 6, 10
    sizes, held = [], set()
    for j in range(1, most + 1):
        for slices in {max(2, nw * (j - 1) + 1), max(2, nw * j)}:
            nb = ((slices - 1) * 64 - 5) * E + 1 - E % 2
            assert _slices(prec, nb, rt * rp) == slices
            held.add(-(-slices // nw))
            sizes.append(nb)
    assert held == set(range(2 if nw == 1 else 1, most + 1))
    lay = T.Layout(NT, NP, np.concatenate([[0], np.cumsum(sizes)]))
    rng = synth.rng(1000 * most + threads)
    tuck = []
    for g, nb in enumerate(sizes):
        pair = []
        for a in range(2):
            core, ut, up, ub = synth.synthetic_tucker(rng, NT, NP, nb, rt, rp, min(nb, 5 + (2 * g + a) % 9))
            pair.append((core, (ut, up, ub)))
        tuck.append(pair)
    h = T.fmm_tucker_create(lay)
    try:
        for g, pair in enumerate(tuck):
            for a, (core, (ut, up, ub)) in enumerate(pair):
                T.fmm_tucker_set_group(h, g, a, core, ut, up, ub)
        ar = arena(T.fmm_tucker_storage_bytes(h, prec)[1])
        T.fmm_tucker_upload(h, prec, ar)
        for nrhs in (1, 2, 4, 5):
            banner("stream wide prec=%d threads=%d most=%d split=%d nrhs=%d" % (prec, threads, most, split, nrhs))
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
