"""The assembly-level checks of test_isa_hazards.py for the masked-edge GEMM flavours (CPU only)."""
import os
import re

from test_isa_hazards import ROOT, _assembly, scan

CSRC = os.path.join(ROOT, "paper_2204_06514_amd", "csrc")


def test_edge_gemm_loads_are_waited_for(tmp_path):
    n, bad = scan(_assembly(tmp_path, os.path.join(CSRC, "kernels_gemm_edge.hip")))
    assert n >= 36, n   # twelve flavours at three tile classes
    assert not bad, {k: v[:3] for k, v in bad.items()}


def test_deep_gemm_assembly_blocks(tmp_path):
    """The blocks hold only loads into LDS, waits and barriers, and every wait in front of a barrier leaves zero to three whole
    slabs' loads in flight (a slab: three instructions a wave at 128 x 64, two at 64 x 64).  How many are in flight where is not
    followed here: whole and cut slabs are requested on two branches, which a walk in straight line counts both."""
    text = _assembly(tmp_path, os.path.join(CSRC, "kernels_gemm_deep.hip"))
    n, bad = scan(text, r"_ZN3fax16gemm_deep_kernel")
    assert n == 24, n   # twelve flavours at two tile classes
    assert not [p for v in bad.values() for p in v if "possibly in flight" not in p]
    n, bad = scan(text, r"_ZN3fax21gemm_deep_pair_kernel")
    assert n == 16, n   # two tile classes and two flavours of either product
    assert not [p for v in bad.values() for p in v if "possibly in flight" not in p]
    for k in re.split(r"\n(?=_ZN3fax(?:16gemm_deep|21gemm_deep_pair)_kernel[^\n]*:\s)", text)[1:]:
        name = k.split(":")[0]
        if "pair" in name:
            slabs = {3 if t == "128" else 2 for t in re.findall(r"Li(128|64)E", name)}
        else:
            slabs = {3 if "ILi128ELi64E" in name else 2}
        waits = re.findall(r"#ASMSTART\s+s_waitcnt vmcnt\((\d+)\)\s+s_barrier\s", k)
        assert set(waits) == {str(i * slab) for i in range(4) for slab in slabs}, waits


def test_loss_gemm_loads_are_waited_for_and_nothing_goes_to_scratch(tmp_path):
    text = _assembly(tmp_path, os.path.join(CSRC, "kernels_gemm_lse.hip"))
    n, bad = scan(text)
    assert n == 3, n   # whole and masked 256 x 256 tiles, the strip's 256 x 128
    assert not bad, {k: v[:3] for k, v in bad.items()}
    assert not re.search(r"^\s*scratch_", text, re.M)


def test_grouped_gemm_loads_are_waited_for(tmp_path):
    text = _assembly(tmp_path, os.path.join(CSRC, "kernels_gemm_group.hip"))
    n, bad = scan(text)
    assert n == 8, n   # two tile classes, whole and masked, stored and added to
    assert not bad, {k: v[:3] for k, v in bad.items()}
    # the same with an input gradient: whatever its width, 256 rows of A in either part, which is what the name of the other kernel says
    text = re.sub(r"_ZN3fax23gemm_group_input_kernelI(?!Li256ELi)", "_ZN3fax23gemm_group_input_kernelILi256ELi", text)
    n, bad = scan(text, r"_ZN3fax23gemm_group_input_kernel")
    assert n == 8, n   # two widths, whole and masked, stored and added to
    assert not bad, {k: v[:3] for k, v in bad.items()}
