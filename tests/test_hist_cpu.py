"""Host side of the sliding-histogram form: which calls take it, that the
configuration reported can be asked for, and what stays refused."""
import ctypes

import pytest

from paper_2507_19926_amd import _lib


# first square window of the form, by type
FIRST = {_lib.MF_U8: 13, _lib.MF_U16: 23, _lib.MF_U32: 21, _lib.MF_F32: 21}


def _resolve(dtype, k, *opt):
    o, r = _lib.options(*opt), _lib.mf_options()
    _lib.check(_lib.lib().mf_query_options(dtype, k, ctypes.byref(o), ctypes.byref(r)))
    return r.variant, r.tile_w, r.tile_h, r.group, r.form, r.rows


@pytest.mark.parametrize("k", list(range(3, 76, 2)))
def test_choice_by_type_and_window(k):
    hist = (_lib.MF_VARIANT_DATA_AWARE, 1, 1, 1, 3, 0)
    for dtype, first in FIRST.items():
        assert (_lib.query_options(dtype, k) == hist) == (k >= first)


def test_reported_configuration_resolves_to_itself():
    for dtype, first in FIRST.items():
        for k in (first, 75):
            v, tw, th, g, f, r = _lib.query_options(dtype, k)
            assert _resolve(dtype, k, v, (tw, th), g, f, r) == (v, tw, th, g, f, r)


def test_refused():
    for dtype, k, o in ((_lib.MF_U8, 11, (_lib.MF_VARIANT_DATA_AWARE, None, 0, 3)),
                        (_lib.MF_U16, 17, (_lib.MF_VARIANT_DATA_AWARE, None, 0, 3)),
                        (_lib.MF_U8, 25, (_lib.MF_VARIANT_AUTO, None, 0, 3)),
                        (_lib.MF_U8, 17, (_lib.MF_VARIANT_OBLIVIOUS, None, 0, 3)),
                        (_lib.MF_U8, 25, (_lib.MF_VARIANT_DATA_AWARE, (2, 1), 0, 3)),
                        (_lib.MF_U8, 25, (_lib.MF_VARIANT_DATA_AWARE, (1, 1), 2, 3))):
        with pytest.raises(_lib.MfError):
            _resolve(dtype, k, *o)
