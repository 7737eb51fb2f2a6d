"""The single-multiply-add forms of the requantisation (requant_f, requant_top):
where the host admits a layer to them they equal the oracle's requantisation on
accumulators across int32, and their arithmetic is defined modulo 2^32, since a
product may leave int32 where its sum with the rounding term does not.  Host
computation only."""
import os
import re
import shutil
import subprocess
import tempfile

import numpy as np
import pytest

from oracle import oracle as O
from paper_2603_25260_amd import build as B
from paper_2603_25260_amd import lpcc
from tests.test_requant_bounds import accumulators, param_sets, s24, wrap32


def more_sets():
    """Layers as models have them: ReLU, identity and PReLU over the shifts the
    forms admit, zero points, multipliers of 31 bits (admitted nowhere)."""
    rng = np.random.default_rng(5)
    sets = []
    for r in (0, 1, 8, 12, 16, 20, 23, 24, 25, 30, 31):
        for _ in range(6):
            m = int(2 ** r * 2.0 ** rng.uniform(-14, 1)) + 1
            z = int(rng.integers(-128, 128))
            sets += [(m, m, r, z), (m, 0, r, z), (m, m >> 2, r, z), (m, m, r, 0)]
    sets += [(1 << 30, 1 << 30, 40, 0), ((1 << 30) + 12345, 0, 41, -3)]
    return sets


def form_f(a, p, r):
    """requant_f: no clamp of the output follows."""
    a = min(max(a, p["f_lo"]), p["f_hi"])
    return wrap32(s24(a) * s24(p["f_m"]) + p["f_rnd"]) >> r


def form_top(a, p):
    """requant_top with both selections of the multiplier: the scaled output."""
    a = min(max(a, p["f_lo"]), p["f_hi"])
    return wrap32(s24(a) * s24(p["t_mn"] if p["rqt"] == 2 and a < 0 else p["t_m"]) + p["t_rnd"])


@pytest.mark.parametrize("m_pos,m_neg,r,z", param_sets() + more_sets())
def test_admitted_forms_equal_oracle(m_pos, m_neg, r, z):
    p = lpcc.requant_fast(m_pos, m_neg, r, z)
    _, _, a_lo, a_hi, _ = lpcc.requant_bounds(m_pos, m_neg, r, z)
    acc = accumulators(a_lo, a_hi, np.random.default_rng(m_pos * 3 + m_neg + r * 17 + z + 1000))
    want = O.requant(acc, m_pos, m_neg, r, z).astype(np.int64)
    if p["rqf"]:
        assert [form_f(int(a), p, r) for a in acc] == want.tolist()
    if p["rqt"]:
        top = np.array([form_top(int(a), p) for a in acc], np.int64)
        assert np.array_equal(top >> 24, want)
        for res in (-128, -1, 0, 7, 127):  # a residual added to the scaled output, saturating
            sat = np.clip(top + (res << 24), -(1 << 31), (1 << 31) - 1)
            assert np.array_equal(sat >> 24, np.clip(want + res, -128, 127))


def test_which_layers_are_admitted():
    """The seeded layers of every width, with one multiplier and with two; a
    logit layer whose product alone leaves int32; and what needs 64 bits."""
    for C in (16, 32, 64):
        m = int(int((1 << 24) / (73.6 * np.sqrt(C))) * 0.75)
        for neg, kind in ((m, (1, 1)), (0, (1, 1)), ((m * 64) >> 8, (0, 2))):
            p = lpcc.requant_fast(m, neg, 24, 0)
            assert (p["rqf"], p["rqt"]) == kind, (C, neg)
    m = int(int((1 << 24) / (73.6 * np.sqrt(32))) * 0.75)
    p = lpcc.requant_fast(m, m, 24, -8)
    assert (p["rqf"], p["rqt"]) == (1, 1)
    assert p["f_hi"] * p["f_m"] >= 1 << 31 > p["f_hi"] * p["f_m"] + p["f_rnd"]
    for args in ((1 << 23, 1 << 23, 1, 0), (1 << 30, 1 << 30, 40, 0), (100, 100, 31, 0)):
        p = lpcc.requant_fast(*args)
        assert (p["rqf"], p["rqt"]) == (0, 0), args


def test_rejects_parameters_outside_the_blob_format():
    for args in ((-1, 0, 5, 0), (0, -1, 5, 0), (1, 1, 63, 0), (1, 1, -1, 0), (1, 1, 5, 128), (1, 1, 5, -129)):
        with pytest.raises(lpcc.LpccError):
            lpcc.requant_fast(*args)


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
