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


class Plan(ctypes.Structure):
    """Mirror of the library's internal MfmaPlan."""
    _fields_ = [("tile", ctypes.c_int), ("bm", ctypes.c_int), ("bn", ctypes.c_int), ("splitk", ctypes.c_int), ("kper", i64),
                ("workspace_bytes", ctypes.c_uint64), ("planes_only", ctypes.c_bool), ("mask_given", ctypes.c_bool),
                ("split_optional", ctypes.c_bool)]


def plan(g, N, pieces, flags=0):
    return internal("_ZN4lrbi9plan_mfmaERKNS_4GeomEjlb", Plan, vp, ctypes.c_uint32, i64, ctypes.c_bool)(ctypes.addressof(g), flags, N, pieces)


PIPE, PIPE256 = 14, 15


@pytest.mark.parametrize("m,n,c,N,pieces,tile,slices", [
    # the 32-column panel kernel, two workgroups per compute unit
    (16640, 4096, 512, 5, False, 11, 2), (16640, 4096, 512, 30, False, 11, 2), (12800, 4096, 512, 7, False, 11, 3),
    (11008, 8192, 512, 13, False, 11, 3), (4224, 9216, 512, 5, False, 11, 8), (4224, 9216, 512, 18, False, 11, 7),
    # tile widths of 64 (2 j + 1), X not in 16-byte pieces: the general kernel runs, two workgroups per compute unit
    (16640, 4096, 64, 36, False, PIPE, 2), (5504, 4608, 192, 389, False, PIPE, 2), (4224, 9216, 192, 389, False, PIPE, 2),
    # the pipelined kernel, one workgroup per compute unit, and the panel kernel that stands in for it
    (5504, 4608, 192, 392, True, PIPE, 1), (5504, 4608, 512, 389, False, PIPE, 1), (4224, 9216, 512, 128, True, PIPE, 7),
])
def test_slices_of_panel_plans(m, n, c, N, pieces, tile, slices):
    p = plan(geom(m, n, 128, c, 16), N, pieces)
    assert (p.tile, p.splitk) == (tile, slices)
    assert p.workspace_bytes == (slices * m * (-(-N // 4) * 4) * 4 if slices > 1 else 0)


def given(g, N):
    p = Plan()
    fn = internal("_ZN4lrbi10plan_givenERKNS_4GeomEjlPNS_8MfmaPlanE", ctypes.c_bool, vp, ctypes.c_uint32, i64, vp)
    return p if fn(ctypes.addressof(g), 0, N, ctypes.addressof(p)) else None


# sizes at which both ways were timed: the decode first (True) or the general kernel
@pytest.mark.parametrize("args,N,first", [
    ((16000, 400, 256, 256, 16), 1000, False), ((8000, 400, 128, 576, 32), 1000, False),  # cut off, lined up, short rows: 44 us against 50
    ((8000, 520, 64, 64, 8), 1000, False), ((4000, 392, 192, 128, 16), 200, False), ((300, 2000, 300, 256, 33), 400, False),
    ((292, 3040, 292, 64, 64), 472, False), ((1714, 448, 192, 320, 55), 432, False), ((2000, 2000, 576, 512, 145), 200, False),
    ((16000, 4096, 64, 64, 8), 64, False), ((2000, 648, 300, 300, 8), 200, False), ((8000, 392, 100, 100, 8), 1000, False),
    ((16000, 1600, 256, 256, 16), 2000, True), ((1000, 4096, 64, 64, 8), 1000, True), ((960, 640, 192, 128, 16), 2000, True),
    ((3000, 3000, 300, 300, 8), 512, True), ((12000, 12000, 300, 300, 8), 40, True), ((2304, 2048, 576, 512, 145), 128, True),
    ((8000, 1000, 100, 100, 8), 1000, True), ((14034, 6520, 100, 256, 8), 80, True), ((5248, 512, 64, 128, 16), 1568, True),
    ((802, 1448, 100, 128, 64), 800, False),
    ((4096, 4096, 256, 256, 16), 1024, False), ((4096, 4096, 128, 192, 16), 1024, False),  # lined up: the mask formed in the kernel
])
def test_mask_decoded_first_where_it_pays(args, N, first):
    p = given(geom(*args), N)
    assert (p is not None) is first
    if p is not None:
        assert p.mask_given and p.tile == PIPE and p.kper % 128 == 0 and p.splitk * p.kper >= args[1] > (p.splitk - 1) * p.kper


# sizes at which both forms of the weight gradient were timed: 256 x 256 tiles (True) or 128 x 128
@pytest.mark.parametrize("m,n,N,wide", [
    (4096, 4096, 128, True), (3840, 4096, 1024, True), (2304, 4096, 1024, True), (2048, 4096, 1024, False), (4096, 3328, 256, False),
    (8192, 4096, 128, False), (8192, 4096, 256, False), (8192, 4096, 512, True), (6912, 4096, 384, True),
    (8192, 8192, 128, False), (8192, 8192, 256, False), (8192, 8192, 512, True), (12800, 12800, 256, False),
    (9216, 9216, 128, False), (9216, 9216, 512, False), (9216, 9216, 1024, True), (4096, 9216, 512, False),
])
def test_gradient_in_wide_tiles(m, n, N, wide):
    fn = internal("_ZN4lrbi12grad256_winsERKNS_4GeomEl", ctypes.c_bool, vp, i64)
    assert fn(ctypes.addressof(geom(m, n, 256, 256, 16)), N) is wide
    assert fn(ctypes.addressof(geom(m, n, 128, 64, 20)), N) is wide


@pytest.mark.parametrize("m,n,N,wide", [(8192, 4096, 128, True), (8192, 8192, 256, True), (12288, 4096, 384, True), (9216, 9216, 256, False)])
def test_gradient_in_wide_tiles_of_many_ranks(m, n, N, wide):
    fn = internal("_ZN4lrbi12grad256_winsERKNS_4GeomEl", ctypes.c_bool, vp, i64)
    assert fn(ctypes.addressof(geom(m, n, 128, 64, 40)), N) is wide
