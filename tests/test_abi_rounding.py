"""The rounding probe refuses bad arguments before it enqueues anything."""


def test_rounding_probe_validation():
    from paper_2005_06671_amd import _lib as L
    f = L.lib().ss_probe_rounding
    for args in ((0, None), (0, 0x200004), (-91, 0x200000), (91, 0x200000)):
        assert f(*args, None) == L.SS_ERR_INVALID_ARG, args
