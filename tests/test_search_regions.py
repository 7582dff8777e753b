"""The workspace regions that the threshold searches borrow, on the host: each is
large enough for what the search keeps there, at every grid of tiles."""

from __future__ import annotations

import ctypes

import pytest


class _Geom(ctypes.Structure):  # spamm_host::Geom
    _fields_ = [(f, ctypes.c_int64) for f in ("n", "bdim", "side", "ntiles", "pyr")] + [
        (f, ctypes.c_int32) for f in ("leaf", "lv", "nwords")
    ]


@pytest.mark.parametrize("leaf", [16, 32, 64, 128])
def test_borrowed_regions_hold_what_the_searches_keep(leaf):
    from paper_2103_13042_amd import binding

    lib = binding.library()
    make_geom = getattr(lib, "_ZN10spamm_host9make_geomEliPNS_4GeomE")
    make_geom.argtypes = [ctypes.c_int64, ctypes.c_int32, ctypes.c_void_p]
    make_geom.restype = ctypes.c_bool
    regions = getattr(lib, "_ZN10spamm_host14search_regionsERKNS_4GeomEPNS_13SearchRegionsE")
    regions.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
    regions.restype = ctypes.c_bool
    geom, out = _Geom(), (ctypes.c_int64 * 16)()
    bad = []
    for bdim in range(1, 1025):
        for n in {(bdim - 1) * leaf + 1, bdim * leaf - leaf // 2, bdim * leaf}:
            assert make_geom(n, leaf, ctypes.byref(geom)) and geom.bdim == bdim
            if not regions(ctypes.byref(geom), out):
                bad.append((n, bdim))
    assert not bad, bad
