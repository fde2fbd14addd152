"""The short forms of reciprocal, root and quotient in the ray and view set-up and in the resample
round as the general ones do: every mantissa, at exponents over the range they are let through
(origins and suns give reciprocals between 1e-30 and 1e30, heights and lengths much less), and
quotients of which half lie next to the middle of two neighbouring numbers.  Any other rounding
would show on both sides of the tests that compare paths, as all of them set rays up this way."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def L():
    from paper_2005_06671_amd import _lib
    _lib.lib()
    return _lib


@pytest.mark.parametrize("exponents", [(-90, -61), (-40, -24), (-13, -8), (-3, -2), (-1, 0), (1, 2), (7, 12),
                                       (21, 38), (60, 90)])
def test_short_forms_round_as_the_general_ones(L, exponents):
    counts = torch.zeros(5, dtype=torch.int64, device="cuda")
    for e in exponents:
        print("rounding", e, flush=True)
        assert L.lib().ss_probe_rounding(e, counts.data_ptr(), None) == L.SS_OK
        torch.cuda.synchronize()
        assert counts.tolist() == [0, 0, 0, 0, 0], e
