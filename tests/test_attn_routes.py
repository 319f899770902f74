"""Which form bf16 attention takes (host only): on both sides of every line, and for the sizes of the GPU tests that are about the forms."""
import pytest

import paper_2204_06514_amd as fax
from test_gpu_attn_forms import CASES

SCALAR, F32, WHOLE, EDGE = fax.FAX_ATTENTION_SCALAR, fax.FAX_ATTENTION_F32, fax.FAX_ATTENTION_MFMA, fax.FAX_ATTENTION_EDGE


def _route(dtype, *size):
    r = fax.fax_attention_route(dtype, *size)
    return r.form, r.groups, r.waves, r.joint


# as in CASES, case by case: form, groups, waves, one launch
FORMS = ([(EDGE, 4, 1, 1)] * 4 + [(WHOLE, 4, 1, 1), (EDGE, 4, 1, 1)] * 2 + [(WHOLE, 4, 1, 1)]
         + [(EDGE, 2, 2, 1), (EDGE, 2, 2, 0), (WHOLE, 2, 2, 1), (EDGE, 2, 2, 1), (EDGE, 2, 2, 1)]
         + [(WHOLE, 2, 2, 0), (EDGE, 2, 2, 0)]
         + [(WHOLE, 1, 4, 0), (EDGE, 1, 4, 0), (EDGE, 1, 4, 0)]
         + [(EDGE, 2, 2, 1)] * 3 + [(WHOLE, 2, 2, 1)] * 2 + [(EDGE, 2, 2, 1)] * 2 + [(EDGE, 2, 2, 0), (WHOLE, 2, 2, 0)]
         + [(EDGE, 2, 4, 0), (WHOLE, 2, 4, 0)] * 2
         + [(WHOLE, 1, 4, 0), (EDGE, 1, 4, 0)])


def test_the_gpu_tests_run_the_forms_they_are_about():
    assert len(FORMS) == len(CASES)
    for size, form in zip(CASES, FORMS):
        assert _route(fax.FAX_BF16, *size) == form, size
    # every kernel there is: whole and masked edges, 64, 96 and 128 wide, in each form; and both backward launches where there is a choice
    seen = {(f[0], 64 if s[3] <= 64 else 96 if f[0] == EDGE and s[3] <= 96 else 128) + f[1:] for s, f in zip(CASES, FORMS)}
    narrow = {(form, 64) + k for form in (WHOLE, EDGE) for k in ((4, 1, 1), (2, 2, 1), (2, 2, 0), (1, 4, 0))}
    wide = {(form, w) + k for form, w in ((WHOLE, 128), (EDGE, 96)) for k in ((2, 2, 1), (2, 4, 0), (1, 4, 0))}
    assert narrow | wide | {(WHOLE, 128, 2, 2, 0), (EDGE, 128, 2, 2, 1), (EDGE, 128, 2, 2, 0)} <= seen


@pytest.mark.parametrize("size,form", [
    ((1, 8160, 1, 64), (EDGE, 4, 1, 1)), ((1, 8192, 1, 64), (WHOLE, 4, 1, 0)), ((1, 8193, 1, 64), (EDGE, 2, 2, 1)),  # 256 tiles of 32 rows; two rounds, one a CU
    ((1, 512, 128, 64), (WHOLE, 2, 2, 0)), ((1, 513, 114, 40), (EDGE, 1, 4, 0)),        # 1024 tiles of 64
    ((1, 64, 511, 64), (EDGE, 2, 2, 1)), ((1, 64, 512, 64), (EDGE, 2, 2, 0)),           # two rounds of workgroups, two a CU
    ((1, 64, 384, 80), (EDGE, 2, 2, 0)), ((1, 64, 385, 80), (EDGE, 2, 4, 0)),           # 384 tiles of 64
    ((1, 64, 170, 128), (EDGE, 2, 2, 1)), ((1, 64, 171, 128), (EDGE, 2, 2, 0)),         # two rounds, one a CU
    ((1, 128, 400, 128), (WHOLE, 2, 4, 0)), ((1, 128, 401, 128), (WHOLE, 1, 4, 0))])    # 400 tiles of 128
def test_lines_between_the_forms(size, form):
    assert _route(fax.FAX_BF16, *size) == form


def test_other_kernels():
    assert _route(fax.FAX_BF16, 4, 1000, 16, 60) == _route(fax.FAX_BF16, 4, 1000, 16, 256) == (SCALAR, 0, 0, 0)
    assert _route(fax.FAX_F32, 4, 512, 16, 64) == (F32, 0, 0, 0) and _route(fax.FAX_F32, 4, 1000, 16, 30) == (SCALAR, 0, 0, 0)
    for bad in ((7, 1, 1, 1, 64), (fax.FAX_BF16, 0, 1, 1, 64), (fax.FAX_BF16, 1, 1, 1, 0)):
        with pytest.raises(fax.FaxError):
            _route(*bad)
