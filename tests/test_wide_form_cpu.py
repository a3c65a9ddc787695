"""xtm_wide_form checks its arguments before it looks at a handle."""
import ctypes

import pytest


@pytest.mark.parametrize("lat,batch,backward,out", [(0, 0, 0, True), (256, 256, 0, True),
                                                    (256, 0, 0, False), (0, 256, 1, True)])
def test_arguments(lat, batch, backward, out):
    import paper_2310_00317_amd as P
    state = ctypes.c_int32()
    code = P.lib().xtm_wide_form(lat or None, batch or None, backward,   # never dereferenced
                                 ctypes.byref(state) if out else None, None)
    assert code == -1
