"""Which kernel a batch's runs take, as af_batch_on_strips tells it (no GPU
needed): strips for grids of ordinary shape, tiles for grids of few columns and
many rows, and tiles from the moment a variant is set."""
import ctypes as C

import pytest

from paper_2609_29081_amd import af


def batch(sizes, precision):
    p = af.Params()
    assert af.lib().af_default_params(C.byref(p)) == af.AF_OK
    ctxs = (C.c_void_p * len(sizes))()
    for i, (p.n1, p.n2) in enumerate(sizes):
        p.precision = precision
        h = C.c_void_p()
        assert af.lib().af_init_grid(C.byref(p), C.byref(h)) == af.AF_OK
        ctxs[i] = h.value
    b = C.c_void_p()
    assert af.lib().af_batch_create(ctxs, len(sizes), C.byref(b)) == af.AF_OK
    return b, ctxs


@pytest.mark.parametrize("precision", [af.PREC_FP64, af.PREC_MIXED])
def test_on_strips(precision):
    L = af.lib()
    for sizes, strips in (([(400, 200)], 1), ([(64, 32)] * 20, 1), ([(4, 30000)] * 8, 0)):
        b, ctxs = batch(sizes, precision)
        assert L.af_batch_on_strips(b) == strips, sizes
        v = L.af_batch_variant(b)
        assert L.af_batch_set_variant(b, v) == af.AF_OK
        assert L.af_batch_on_strips(b) == 0 and L.af_batch_variant(b) == v
        L.af_batch_destroy(b)
        for c in ctxs:
            L.af_destroy(C.c_void_p(c))
    assert L.af_batch_on_strips(None) == -1
