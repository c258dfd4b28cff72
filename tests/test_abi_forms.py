"""Argument checks of the form queries, without a GPU."""
import ctypes


def test_form_queries_refuse_null():
    import paper_2603_23343_amd as P

    f = ctypes.c_int(7)
    for fn in (P.lib.pcg_get_form, P.lib.pcg_batch_get_form):
        assert fn(None, ctypes.byref(f)) == P.PCG_E_ARG
        assert P.pcg_last_error()
    assert f.value == 7
