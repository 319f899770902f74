"""Which form bf16 attention takes, forward and backward (host only): on both sides of every line, and for the sizes of the GPU tests that are about the
forms."""
import pytest

import paper_2204_06514_amd as fax
from test_gpu_attn_forms import CASES

SCALAR, F32, WHOLE, EDGE = fax.FAX_ATTENTION_SCALAR, fax.FAX_ATTENTION_F32, fax.FAX_ATTENTION_MFMA, fax.FAX_ATTENTION_EDGE


def _route(dtype, *size):
    """kernel, forward form, backward form: groups and waves as one number, j where dQ and dK/dV share a launch"""
    r = fax.fax_attention_route(dtype, *size)
    return r.form, "%d%d" % (r.groups, r.waves), "%d%d%s" % (r.bwd_groups, r.bwd_waves, "j" if r.joint else "")


# as in CASES, row by row
FORMS = [
    (EDGE, "14", "22j"), (EDGE, "14", "22j"), (EDGE, "14", "22j"), (EDGE, "22", "22j"), (WHOLE, "22", "22j"), (EDGE, "41", "41j"), (WHOLE, "41", "41j"),
    (EDGE, "41", "41j"), (WHOLE, "41", "41j"),
    (EDGE, "14", "14"), (EDGE, "14", "14"), (WHOLE, "22", "22j"), (EDGE, "22", "22j"), (EDGE, "22", "22j"),
    (WHOLE, "22", "22"), (EDGE, "22", "22"),
    (WHOLE, "14", "14"), (EDGE, "14", "14"), (EDGE, "14", "14"),
    (EDGE, "14", "22j"), (EDGE, "14", "22j"), (EDGE, "22", "22j"), (WHOLE, "22", "22j"), (WHOLE, "22", "22j"), (EDGE, "22", "22j"), (EDGE, "22", "22j"),
    (EDGE, "24", "24"), (WHOLE, "24", "22"),
    (EDGE, "14", "14"), (WHOLE, "14", "14"), (EDGE, "14", "14"), (WHOLE, "14", "14"),
    (WHOLE, "14", "14"), (EDGE, "14", "14"),
    (EDGE, "41", "41j"), (EDGE, "41", "41j"), (WHOLE, "24", "24"), (EDGE, "24", "24"), (EDGE, "24", "24"), (EDGE, "22", "22"), (EDGE, "22", "22"), (EDGE, "14", "14")]


def test_the_gpu_tests_run_the_forms_they_are_about():
    assert len(FORMS) == len(CASES)
    for size, form in zip(CASES, FORMS):
        assert _route(fax.FAX_BF16, *size) == form, size
    # every kernel there is: whole and masked edges, 64, 96 and 128 wide, in each form, forward and backward
    width = lambda s, f: 64 if s[3] <= 64 else 96 if f[0] == EDGE and s[3] <= 96 else 128  # noqa: E731
    seen = {(f[0], width(s, f), d, f[1 + d]) for s, f in zip(CASES, FORMS) for d in (0, 1)}
    kinds = [(WHOLE, 64), (EDGE, 64), (WHOLE, 128), (EDGE, 96), (EDGE, 128)]
    want = {(k, w, 0, f) for k, w in kinds for f in (("14", "22", "41") if w == 64 else ("14", "22", "24"))}
    want |= {(k, w, 1, f) for k, w in kinds for f in (("14", "22", "22j", "41j") if w == 64 else ("14", "22", "22j", "24"))}
    assert want <= seen, want - seen


@pytest.mark.parametrize("d,dh,lines", [
    # sequence length: (heads up to which, form) ..., then the last form
    (0, 64, {64: "14", 65: [(200, "22"), "14"], 128: [(200, "22"), "14"], 129: [(51, "41"), (266, "22"), "14"], 256: [(32, "41"), (200, "22"), "14"],
             257: [(28, "41"), (204, "22"), "14"], 2048: [(4, "41"), (32, "22"), "14"]}),
    (1, 64, {64: [(256, "22j"), "14"], 65: [(159, "22j"), (200, "22"), "14"], 129: [(28, "41j"), (129, "22j"), (266, "22"), "14"], 256: [(18, "41j"), (97, "22j"), (200, "22"), "14"],
             257: [(16, "41j"), (102, "22j"), (204, "22"), "14"], 385: [(19, "41j"), (73, "22j"), (146, "22"), "14"], 2048: [(4, "41j"), (15, "22j"), (32, "22"), "14"]}),
    (0, 128, {64: "14", 65: [(128, "22"), "14"], 129: [(85, "22"), (128, "24"), "14"], 384: [(42, "22"), (85, "24"), "14"], 385: [(36, "22"), (75, "24"), "14"],
              640: [(25, "22"), (60, "24"), "14"], 641: [(23, "22"), (88, "24"), "14"], 705: [(34, "22"), (88, "24"), "14"], 2048: [(13, "22"), (33, "24"), "14"]}),
    (1, 80, {32: [(128, "22j"), "14"], 64: [(85, "22j"), "14"], 65: [(100, "22j"), (128, "24"), "14"], 128: [(83, "22j"), (128, "24"), "14"], 129: [(68, "22j"), (128, "24"), "14"],
             256: [(50, "22j"), (57, "22"), (128, "24"), "14"], 448: [(28, "22j"), (33, "22"), (75, "24"), "14"], 449: [(26, "22j"), (39, "22"), (75, "24"), "14"],
             641: [(18, "22j"), (28, "22"), (66, "24"), "14"], 2048: [(6, "22j"), (9, "22"), (25, "24"), "14"]}),
    (1, 128, {128: [(100, "22j"), (128, "22"), "14"], 256: [(50, "22j"), (57, "22"), (128, "24"), "14"], 512: [(25, "22j"), (37, "22"), (64, "24"), "14"],
              640: [(20, "22j"), (30, "22"), (51, "24"), "14"], 1024: [(12, "22j"), (18, "22"), (40, "24"), "14"], 2048: [(6, "22j"), (9, "22"), (20, "24"), "14"],
              2176: [(5, "22j"), (8, "22"), (23, "24"), "14"]})])
def test_lines_between_the_forms(d, dh, lines):
    for S, forms in lines.items():
        if isinstance(forms, str):
            assert {_route(fax.FAX_BF16, 1, S, h, dh)[1 + d] for h in (1, 7, 100, 3000)} == {forms}, S
            continue
        for (most, form), after in zip(forms[:-1], [f[1] for f in forms[1:-1]] + [forms[-1]]):
            assert _route(fax.FAX_BF16, 1, S, most, dh)[1 + d] == form, (S, most)
            assert _route(fax.FAX_BF16, 1, S, most + 1, dh)[1 + d] == after, (S, most)
            assert _route(fax.FAX_BF16, most, S, 1, dh) == _route(fax.FAX_BF16, 1, S, most, dh)


def test_other_kernels():
    none = "00"
    assert _route(fax.FAX_BF16, 4, 1000, 16, 60) == _route(fax.FAX_BF16, 4, 1000, 16, 256) == (SCALAR, none, none)
    assert _route(fax.FAX_F32, 4, 512, 16, 64) == (F32, none, none) and _route(fax.FAX_F32, 4, 1000, 16, 30) == (SCALAR, none, none)
    for bad in ((7, 1, 1, 1, 64), (fax.FAX_BF16, 0, 1, 1, 64), (fax.FAX_BF16, 1, 1, 1, 0)):
        with pytest.raises(fax.FaxError):
            _route(*bad)
