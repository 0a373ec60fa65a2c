"""The allocation-free forward refuses, before any HIP call, a column-owning
variant that would wait on words in the array that all its calls share."""
import ctypes

import numpy as np

FAKE = 1 << 20


def test_column_owning_variants_are_refused():
    import paper_2403_06931_amd as P
    from paper_2403_06931_amd import _lib as L
    h = np.array([300, 70], np.int32)
    cols = [v for v in range(P.sdtw_variant_count()) if P.sdtw_variant_info(v)[0] == 1]
    assert cols
    p = ctypes.c_void_p
    for v in cols:
        rc = L.lib.sdtw_forward_noalloc(p(FAKE), p(h.ctypes.data), p(FAKE), h.size, p(FAKE), 5000,
                                        0, p(FAKE), p(FAKE), p(0), 0, v, 0, p(0))
        assert rc == L.SDTW_ERR_WORKSPACE, L.status_string(rc)
