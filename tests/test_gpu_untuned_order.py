"""Untuned matrix-core calls use one of the angular orders that the tuner offers, so that a tuned
call cannot lose to an untuned one: their results are those of a forced order, bit for bit, on a
layout whose items prefer different orders.
"""
import numpy as np
import pytest

import synth
from gpu_util import dev, host, arena, banner

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2103_05822_amd")


@pytest.mark.parametrize("prec", [T.FMM_C128, T.FMM_C64, T.FMM_BF16X3], ids=["c128", "c64", "bf16x3"])
@pytest.mark.parametrize("slim", [4, 40])  # groups of the second kind among 44
def test_untuned_order_is_offered(prec, slim):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nrhs, n = 6, 44
    cd = np.complex128 if prec == T.FMM_C128 else np.complex64
    lay = T.Layout(7, 11, 40 * np.arange(n + 1))
    rng = synth.rng(slim)
    h = T.fmm_tucker_create(lay)
    try:
        for g in range(n):
            rt = 1 if g < slim else 6  # rank 1: phi first takes a quarter of the products
            for a in range(2):
                T.fmm_tucker_set_group(h, g, a, *synth.synthetic_tucker(rng, 7, 11, 40, rt, 10, 10))
        ar = arena(T.fmm_tucker_storage_bytes(h, prec)[1])
        T.fmm_tucker_upload(h, prec, ar)
        x = dev(synth.complex_normal(rng, (lay.n_basis, nrhs)), cd)
        G = dev(synth.complex_normal(rng, (lay.n_groups, 2, lay.n_dir, nrhs)), cd)

        def run():
            F, V = torch.zeros_like(G), torch.zeros_like(x)
            T.fmm_tucker_pass(h, prec, nrhs, x, F, G, V)
            return host(F).copy(), host(V).copy()

        banner("untuned order prec=%d slim=%d" % (prec, slim))
        untuned = run()
        equal = []
        for order in (0, 1, 2):
            T.fmm_tucker_set_tuned(h, prec, nrhs, path=1, tile_steps=16, rhs_chunk=nrhs, order=order)
            equal.append(all(np.array_equal(a, b) for a, b in zip(untuned, run())))
        print("  equal to orders 0, 1, 2:", equal, flush=True)
        assert equal[0 if slim == 40 else 1]
    finally:
        T.fmm_tucker_destroy(h)
