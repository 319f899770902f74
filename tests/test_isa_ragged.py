"""The assembly-level checks of test_isa_hazards.py for the masked-edge GEMM flavours (CPU only)."""
import os

from test_isa_hazards import ROOT, _assembly, scan

CSRC = os.path.join(ROOT, "paper_2204_06514_amd", "csrc")


def test_edge_gemm_loads_are_waited_for(tmp_path):
    n, bad = scan(_assembly(tmp_path, os.path.join(CSRC, "kernels_gemm_edge.hip")))
    assert n >= 36, n   # twelve flavours at three tile classes
    assert not bad, {k: v[:3] for k, v in bad.items()}
