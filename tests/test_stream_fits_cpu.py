"""The rule that picks the row-streaming kernel (host code, no GPU): its LDS counts what the
kernel declares itself, sizes beyond an int are not taken for small ones, and several right-hand
sides share a read of the factors wherever a workgroup size allows it and units are enough."""
import ctypes

import pytest

T = pytest.importorskip("paper_2103_05822_amd", reason="libtuckfmm.so not built")

LDS = 160 * 1024
STATIC = 16   # the pass kernel's own variable, rounded to its alignment


class TuckMax(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in
                ("nb", "rt", "rp", "rb", "q", "t3", "nt", "np", "row", "slices", "lds", "stage")]


class StreamFit(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("threads", "jmax", "rb", "staged")] + [("lds", ctypes.c_size_t)]


def fits(prec, mx, threads, nrhs, dis=True, units=1000):
    name = "_ZN7tuckfmm11stream_fitsI%sEEbRKNS_7TuckMaxEiiibPNS_9StreamFitE" % ("d" if prec == "c128" else "f")
    fn = getattr(ctypes.CDLL(T.binding.LIB_PATH), name)
    fn.restype = ctypes.c_bool
    fn.argtypes = [ctypes.POINTER(TuckMax), ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_bool, ctypes.POINTER(StreamFit)]
    out = StreamFit()
    return out if fn(ctypes.byref(mx), units, threads, nrhs, dis, ctypes.byref(out)) else None


def multi_threads(mx, units, threads, nrhs):
    fn = ctypes.CDLL(T.binding.LIB_PATH)._ZN7tuckfmm13multi_threadsERKNS_7TuckMaxEiii
    fn.argtypes = [ctypes.POINTER(TuckMax), ctypes.c_int, ctypes.c_int, ctypes.c_int]
    return fn(ctypes.byref(mx), units, threads, nrhs)


def layout(prec, nb, rt, rp, rb, nt, npn, stage=1):
    """One item's maxima, as the library forms them (phi first: the smaller intermediate)."""
    E = 1 if prec == "c128" else 2
    up = lambda v: (v + E - 1) // E * E  # noqa: E731
    ld_u, ld_c = up(nb), up(rt * rp)
    theta, phi = nt * rp * (rt + npn), rt * npn * (rp + nt)
    return TuckMax(nb, rt, rp, rb, rt * rp, nt * rp if theta <= phi else rt * npn, nt, npn, ld_u + ld_c,
                   -(-(ld_u // E) // 64) - (-(ld_c // E) // 64), LDS, stage)


@pytest.mark.parametrize("prec", ["c64", "c128"])
def test_lds_at_the_limit(prec):
    # 512 threads, unstaged: row + inter fill the LDS but for the partial sums and `spare` bytes
    es, real = (8, 4) if prec == "c64" else (16, 8)
    red = 2 * 8 * 16 * real
    total = (LDS - red) // es                 # complex values
    seen = []
    for spare in (0, 8, 16, 24, 32, 64):
        mx = layout(prec, 64, 2, 2, 4, 7, 11, stage=0)
        mx.t3 = 4000
        mx.row = (total - mx.t3) - spare // es // 2 * 2
        f = fits(prec, mx, 512, 1)
        if f is not None:
            assert f.lds + STATIC <= LDS
        seen.append(f is not None)
    assert not seen[0] and seen[-1]


@pytest.mark.parametrize("prec", ["c64", "c128"])
@pytest.mark.parametrize("dis", [True, False])
def test_staging_of_huge_grids(prec, dis):
    # n_theta r_theta = 2^32 + 1: as a 32-bit product it is 1
    mx = layout(prec, 1000, 641, 1, 9, 6700417, 1)
    f = fits(prec, mx, 256, 1, dis)
    assert f is not None and not f.staged


# largest items of boxes of 0.5, 1, 1.5, 2 and 4 wavelengths: n_beta, ranks, grid
BOXES = {0.5: (114, 15, 17, 66, 17, 33), 1.0: (457, 19, 24, 131, 25, 49), 1.5: (1010, 24, 27, 186, 32, 63),
         2.0: (1791, 25, 30, 235, 38, 75), 4.0: (8684, 39, 54, 381, 64, 127)}


@pytest.mark.parametrize("prec", ["c64", "c128"])
@pytest.mark.parametrize("box", sorted(BOXES))
@pytest.mark.parametrize("nrhs", [2, 3, 4, 5, 7])
def test_right_hand_sides_share_a_read(prec, box, nrhs):
    mx = layout(prec, *BOXES[box])
    f1 = fits(prec, mx, 256, 1)
    if f1 is None:  # the general kernel's
        assert (box, prec) == (4.0, "c128")
        return
    t = multi_threads(mx, 2000, 256, nrhs)
    f = fits(prec, mx, t, nrhs, units=2000)
    widest = -(-mx.slices // 8)  # slices a wavefront with 512 threads
    assert (f.rb >= 2) == (widest <= 4) and f.threads >= t
    if f.rb == 1:
        assert t == 256
    # few units: an entry per right-hand side
    assert fits(prec, mx, multi_threads(mx, 16, 256, nrhs), nrhs, units=16).rb == 1
