"""The single-multiply-add forms of the requantisation (requant_f, requant_top):
their arithmetic is defined modulo 2^32, since a product may leave int32 where
its sum with the rounding term does not.  Host computation only."""
import os
import re
import shutil
import subprocess
import tempfile

import pytest

from paper_2603_25260_amd import build as B


@pytest.fixture(scope="module")
def front_end_ir():
    """LLVM IR of the device functions as the front end leaves it."""
    if not os.path.exists(B.HIPCC) and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    src = ('#include "lpcc_internal.h"\n'
           'extern "C" __global__ void k(const lpcc::LayerDev* L, int* o) {\n'
           '  o[0] = lpcc::requant_f(o[0], *L) ^ lpcc::requant_top<false>(o[1], *L) ^ lpcc::requant_top<true>(o[2], *L);\n'
           '}\n')
    flags = [f for f in B.FLAGS if f not in ("-fPIC", "-Wall")]
    with tempfile.TemporaryDirectory() as d:
        hip, out = os.path.join(d, "t.hip"), os.path.join(d, "t.ll")
        with open(hip, "w") as f:
            f.write(src)
        r = subprocess.run([B.HIPCC, *flags, "-I", B.CSRC, "--cuda-device-only", "-S", "-emit-llvm", "-Xclang",
                            "-disable-llvm-passes", "-o", out, hip], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        return open(out).read()


@pytest.mark.parametrize("name", ["requant_fE", "requant_topILb0E", "requant_topILb1E"])
def test_sum_of_product_and_rounding_term_may_wrap(front_end_ir, name):
    """No signed addition or product that the compiler may assume not to
    overflow."""
    body = re.search(r"^define[^\n]*" + name + r".*?^\}", front_end_ir, re.S | re.M).group(0)
    assert "__mul24" in body
    assert not re.findall(r"(?:add|sub|mul) nsw [^\n]*", body)
