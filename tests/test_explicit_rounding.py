"""What the lane walk and the cooperative walk of the hybrid 1D kernels both compute, the log-weight and the
shifted frequency, is written with fma in both: a product and a sum left to the compiler's contraction could be
rounded once in one and twice in the other."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1709_10187_amd", "csrc")


def test_log_weight_and_shift_are_written_with_fma():
    src = open(os.path.join(CSRC, "transport1dh.hip")).read()
    assert not re.search(r"\blw\s*\+=", src)
    assert not re.search(r"rho\s*\*\s*\(double\)xin\s*\+", src)
    assert len(re.findall(r"\blw\s*=\s*fma\(", src)) == 4
    assert len(re.findall(r"fma\(rho, \(double\)xin, sh\)", src)) == 2
