"""The dense kernels with several right-hand sides: the length of their summation chains, and
far-fields at the element's own alignment.

A row of 5700 columns is 11400 products a part.  Summed in 64 chains that meet in a tree, as
64 lanes or 64 accumulators hold them, chains of m = 11400 / 64 random products leave an error
of about u / sqrt(3) sqrt(m / 6) of the result (u = 2^-24 or 2^-53: each addition rounds by
u / sqrt(3) of a partial sum that grows as the square root); one chain leaves eight times
that.  The bound is 2.5 times the value for 64 chains.
"""
import numpy as np
import pytest

import synth
from gpu_util import dev, host, banner

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2103_05822_amd")

CDT = {T.FMM_C128: np.complex128, T.FMM_C64: np.complex64}
UNIT = {T.FMM_C128: 2.0 ** -53, T.FMM_C64: 2.0 ** -24}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)


@pytest.mark.parametrize("prec", [T.FMM_C128, T.FMM_C64], ids=["c128", "c64"])
@pytest.mark.parametrize("nrhs", [2, 5, 8])
@pytest.mark.parametrize("skew", [0, 1])
def test_disaggregation_chains(prec, nrhs, skew):
    lay = T.Layout(38, 75, [0, 5, 38])
    cd, nc = CDT[prec], 2 * lay.n_dir
    rng = synth.rng(40 + nrhs)
    A = synth.complex_normal(rng, (lay.n_basis, nc)).astype(cd)
    gin = synth.complex_normal(rng, (lay.n_groups, nc, nrhs)).astype(cd)
    # `skew` elements in front: a complex64 array that starts 8 bytes past a 16-byte boundary
    flat = dev(np.concatenate([np.full(skew, np.nan, cd), A.ravel()]))
    V = dev(np.full((lay.n_basis, nrhs), np.nan, cd))
    d = T.fmm_dense_create(lay)
    try:
        banner("dense sums prec=%d nrhs=%d skew=%d" % (prec, nrhs, skew))
        T.fmm_dense_disaggregate(d, prec, flat[skew:], nrhs, dev(gin), V)
        got = host(V)
    finally:
        T.fmm_dense_destroy(d)
    wide = np.clongdouble
    ref = np.concatenate([A[lay.offsets[g]:lay.offsets[g + 1]].astype(wide).conj() @ gin[g].astype(wide)
                          for g in range(lay.n_groups)])
    err = float(np.linalg.norm((got - ref).astype(np.complex128)) / np.linalg.norm(ref.astype(np.complex128)))
    bound = 2.5 * UNIT[prec] / np.sqrt(3.0) * np.sqrt(2.0 * nc / 64 / 6.0)
    print("  error %.2e, bound %.2e" % (err, bound), flush=True)
    assert err < bound
