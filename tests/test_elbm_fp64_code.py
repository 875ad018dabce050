"""The out-of-line FP64 root solve of FP32 ELBM sites, compiled by itself: its
code must hold the solve whatever the callers around it look like (a read
through a null pointer would let the compiler drop the iteration and return a
constant)."""
import re
import subprocess

import pytest

from paper_1110_0270_amd import build

SRC = r"""
#include "lbm_collide.h"
using namespace lbm;
__global__ void k(ElbmF64Site s, ElbmF64Result* out) { *out = elbm_alpha_fp64<QQ>(s, 1e-14, 1e-15, 32, 0, 0); }
"""


@pytest.mark.parametrize("q", [3, 9])
def test_the_solve_is_in_the_code(tmp_path, q):
    src = tmp_path / "t.hip"
    src.write_text(SRC.replace("QQ", str(q)))
    r = subprocess.run([build.HIPCC, *build.FLAGS, "-I", build.CSRC, "--offload-device-only", "-S",
                        str(src), "-o", "-"], check=True, capture_output=True, text=True)
    body = re.search(r"^(_ZN3lbm15elbm_alpha_fp64\w+):(.*?)^\.Lfunc_end", r.stdout, re.S | re.M).group(2)
    # one FP64 logarithm per component at least, and a loop around them
    assert len(re.findall(r"\bv_frexp_mant_f64", body)) >= q
    assert re.search(r"s_cbranch", body)
