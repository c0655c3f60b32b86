"""The dense kernels on a layout of more workgroups than one launch holds (2^32 threads): 8.4
million groups of one row and 66 columns, 5 right-hand sides in complex64.  Sampled groups
against their definition in FP64: outer products (one product an entry, 1e-6) and sums of 66
products (1e-5).
"""
import numpy as np
import pytest

from gpu_util import banner

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2103_05822_amd")


def test_more_workgroups_than_a_launch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 80 GB of device memory")
    n, nrhs = (1 << 23) + 5, 5
    lay = T.Layout(3, 11, np.arange(n + 1))
    nc = 2 * lay.n_dir
    gen = torch.Generator(device="cuda").manual_seed(3)
    kw = dict(dtype=torch.complex64, device="cuda")
    A = torch.randn(n, nc, generator=gen, **kw)
    x = torch.randn(n, nrhs, generator=gen, **kw)
    G = torch.randn(n, nc, nrhs, generator=gen, **kw)
    F, V = torch.full_like(G, float("nan")), torch.full_like(x, float("nan"))
    d = T.fmm_dense_create(lay)
    try:
        banner("dense, %d groups" % n)
        T.fmm_dense_aggregate(d, T.FMM_C64, A, nrhs, x, F)
        T.fmm_dense_disaggregate(d, T.FMM_C64, A, nrhs, G, V)
        torch.cuda.synchronize()
    finally:
        T.fmm_dense_destroy(d)
    assert not torch.isnan(V.real).any()
    for r in range(0, n, 1 << 20):
        assert not torch.isnan(F[r:r + (1 << 20)].real).any()
    edge = 1 << 21
    rows = torch.tensor([0, 1, edge - 1, edge, 2 * edge, 3 * edge, 4 * edge - 1, 4 * edge, n - 1], device="cuda")
    a, xs, g = A[rows].to(torch.complex128), x[rows].to(torch.complex128), G[rows].to(torch.complex128)
    f_ref = a[:, :, None] * xs[:, None, :]
    v_ref = (a.conj()[:, :, None] * g).sum(1)
    assert float((F[rows] - f_ref).abs().max() / f_ref.abs().max()) < 1e-6
    assert float((V[rows] - v_ref).abs().max() / v_ref.abs().max()) < 1e-5
