"""Device memory that an in-place handle asks for (host only, nothing is launched).

The workspace has one size at any lattice size, so a caller may keep one for several handles;
the room for the copies of several steps per pass is asked for and bound apart from it.
"""
import ctypes

import pytest

from test_capi_host import _create, _params, capi  # noqa: F401 (fixture)

LAT, WS, HALO = 1 << 40, 1 << 36, 1 << 37   # addresses that are never followed


def handle(capi, **kw):  # noqa: F811
    rc, h = _create(capi, _params(capi, **kw))
    assert rc == 0
    lat, ws, halo = ctypes.c_size_t(), ctypes.c_size_t(), ctypes.c_size_t()
    L = capi.lib()
    assert L.lbmhd_sizes(h, ctypes.byref(lat), ctypes.byref(ws), None, None) == 0
    assert L.lbmhd_halo_bytes(h, ctypes.byref(halo)) == 0
    return h, lat.value, ws.value, halo.value


@pytest.mark.parametrize("nx,ny", [(4096, 4096), (2048, 1500), (64, 48)])
def test_one_workspace_serves_every_handle(capi, nx, ny):  # noqa: F811
    L = capi.lib()
    h0, _, ws0, none = handle(capi)
    h, lat, ws, _ = handle(capi, nx=nx, ny=ny, inplace=1)
    assert ws == ws0 and none == 0
    assert L.lbmhd_bind(h, LAT, lat, None, 0, WS, ws0, None) == 0
    for x in (h0, h):
        assert L.lbmhd_destroy(x) == 0


def test_binding_the_room_for_copies(capi):  # noqa: F811
    L = capi.lib()
    h, lat, ws, halo = handle(capi, nx=4096, ny=4096, inplace=1)
    assert halo > 0 and halo % 256 == 0
    bad = capi.LBMHD_ERR_INVALID_ARG
    assert L.lbmhd_bind_halos(h, HALO, halo) == capi.LBMHD_ERR_NOT_BOUND
    assert L.lbmhd_bind(h, LAT, lat, None, 0, WS, ws, None) == 0
    assert L.lbmhd_bind_halos(h, HALO, halo) == 0
    assert L.lbmhd_bind_halos(h, None, 0) == 0
    assert L.lbmhd_bind_halos(h, HALO, halo - 1) == bad
    assert L.lbmhd_bind_halos(h, HALO + 128, halo) == bad
    assert L.lbmhd_bind_halos(h, LAT + lat - 256, halo) == bad
    assert L.lbmhd_bind_halos(h, WS - halo + 256, halo) == bad
    assert L.lbmhd_bind_halos(None, HALO, halo) == bad
    assert L.lbmhd_halo_bytes(h, None) == bad and L.lbmhd_halo_bytes(None, None) == bad
    assert L.lbmhd_destroy(h) == 0
    # named single steps, FP16 storage and small lattices take none; a buffer is then ignored
    for kw in (dict(steps_per_pass=1), dict(storage=capi.LBMHD_FP16), dict(nx=512, ny=512)):
        h, lat, ws, halo = handle(capi, **{**dict(nx=4096, ny=4096, inplace=1), **kw})
        assert halo == 0
        assert L.lbmhd_bind(h, LAT, lat, None, 0, WS, ws, None) == 0
        assert L.lbmhd_bind_halos(h, HALO, 0) == 0
        assert L.lbmhd_destroy(h) == 0


@pytest.mark.parametrize("nx,ny,rows", [
    (4096, 4096, True), (2048, 1500, True), (16384, 190, True), (257, 11800, True),
    (110000, 28, True), (15600, 193, True), (120000, 33, True), (1600000, 2, False),
    (500000, 6, False), (200000, 16, False)])
def test_copies_stay_below_a_quarter_of_the_lattice(capi, nx, ny, rows):  # noqa: F811
    h, lat, _, halo = handle(capi, nx=nx, ny=ny, inplace=1)
    assert (halo > 0) == rows and 4 * halo <= lat
    assert capi.lib().lbmhd_destroy(h) == 0
