"""Which kernel a call is sent to: the library's own host-side predicates and plans, called without a GPU."""
import ctypes

import pytest

import paper_1905_05686_amd as lrbi

i64, vp = ctypes.c_int64, ctypes.c_void_p


class Geom(ctypes.Structure):
    """Mirror of the library's internal Geom."""
    _fields_ = [("m", i64), ("n", i64)] + [(f, ctypes.c_int32) for f in ("r", "c", "k", "tile_cols", "tile_rows", "ragged", "ipw", "izw")]


def geom(m, n, r, c, k):
    cols, rows = -(-n // c), -(-m // r)
    return Geom(m, n, r, c, k, cols, rows, int(m % r != 0 or n % c != 0), -(-k // 32), 2 * -(-c // 64))


def internal(name, restype, *argtypes):
    fn = getattr(lrbi.load_library(), name)
    fn.restype, fn.argtypes = restype, list(argtypes)
    return fn


def test_geom_mirror():
    make = internal("_ZN4lrbi9make_geomEPK9lrbi_desc", Geom, vp)
    for args in ((4100, 9224, 256, 300, 33), (512, 512, 128, 64, 8)):
        d = lrbi.Desc(*args)
        assert bytes(make(ctypes.addressof(d))) == bytes(geom(*args))


def given_ok(g, ldw, ldx, N, pitch, x=0x1000):
    fn = internal("_ZN4lrbi13pipe_given_okERKNS_4GeomEPKvllll", ctypes.c_bool, vp, vp, i64, i64, i64, i64)
    return fn(ctypes.addressof(g), x, ldw, ldx, N, pitch)


@pytest.mark.parametrize("pitch,ok", [
    (384, True), (1 << 25, True), ((1 << 25) + 16, False), (33818656, False), (1 << 26, False), (1 << 32, False), (1 << 40, False),
])
def test_decoded_mask_offsets_fit_32_bits(pitch, ok):
    """The kernel on a decoded mask addresses the mask rows of a 128-row tile with 32-bit byte offsets."""
    assert given_ok(geom(1200, 3000, 300, 300, 8), 3000, 512, 512, pitch) is ok
    if ok:
        assert 127 * pitch + 16 * ((3000 + 127) // 128) <= 1 << 32
